// Token sampling, retirement/compaction, sibling fork, rollout set-up and the
// group-relative advantage.
#include <algorithm>
#include <type_traits>

#include "rg_device.h"
#include "rg_kernels.h"

namespace {

// ------------------------------------------------------------------ sampling
// Two kernels.  k_sample_slice: block (slice, row) scans one slice of the
// row's vocabulary -- Gumbel scores, running logsumexp of z/T -- and writes
// the slice's (best score, best id, max, sum).  k_sample_pick: one block per
// row combines the slices in order (ties to the lowest id), decides the
// token and writes the outputs.
constexpr int SAMPLE_THREADS = 256;
constexpr float LN2 = 0.693147180559945309f;

// log2(-log2 u) for the 32-bit value x of a token, u = (2 (x >> 9) + 1) 2^-24.
// The Gumbel noise is -ln(-ln u) = -ln 2 log2(-log2 u) - ln(ln 2); the constant,
// the same for every token, is left out of the scores.  Over all 2^23 values of u
// the noise is within 1.81e-6 of its value in 64 bits, 7.3e-8 rms (1.88e-6 and
// 9.6e-8 with the library's logarithm inside, whose instructions bounded the
// slice kernel: 512 rows of 151,936 129 -> 102 us, of which reading the logits
// takes 63): the hardware logarithm keeps its relative error near u = 1 too,
// where -log2 u is ~8.6e-8.
__device__ __forceinline__ float gumbel_log2(uint32_t x) {
  // 1 + (x >> 9) 2^-23 less 1 - 2^-24: exact
  const float u = __uint_as_float((x >> 9) | 0x3F800000u) - 0.999999940395355224609375f;
  return __builtin_amdgcn_logf(-__builtin_amdgcn_logf(u));
}

__global__ void k_gumbel_noise(uint32_t first, int64_t n, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = -LN2 * gumbel_log2((first + (uint32_t)i) << 9);
}

__global__ __launch_bounds__(SAMPLE_THREADS) void k_sample_slice(SampleArgs a) {
  const int r = blockIdx.y;
  if (r >= *a.d_rows) return;
  const int tid = threadIdx.x;
  const int t = *a.d_t;
  const int s = a.act_seq[r];
  const int lrow = a.logits_by_group ? a.seq_grp[s] : r;
  const float* z = a.logits + (int64_t)lrow * a.V;
  const int L = a.forced_len ? a.forced_len[s] : -1;
  const bool mask_eos = L > 0 && t < L - 1;
  const float T = a.temperature;
  const bool unit_T = T == 1.0f;                            // z / 1 == z exactly: skip the division
  const int nb = a.V >> 3;                                  // 8-token Philox blocks
  const int per = (nb + a.n_slices - 1) / a.n_slices;
  const int vb0 = blockIdx.x * per, vb1 = min(nb, vb0 + per);

  // the EOS entry is masked in one 8-token block only
  const int eos_vb = mask_eos ? (a.eos >> 3) : -1, eos_j = a.eos & 7;
  float best = -INFINITY;
  int best_v = 0x7FFFFFFF;
  float m = -INFINITY, sum = 0.f;
  for (int vb = vb0 + tid; vb < vb1; vb += SAMPLE_THREADS) {
    rg_u64x4 c;
    c.v[0] = (uint64_t)vb; c.v[1] = (uint64_t)t; c.v[2] = (uint64_t)s; c.v[3] = 0;
    rg_u64x4 w = rg_philox4x64_10(c, a.seed, RG_TAG_GUMBEL);
    const float4 z0 = *reinterpret_cast<const float4*>(z + vb * 8);
    const float4 z1 = *reinterpret_cast<const float4*>(z + vb * 8 + 4);
    float zt[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
    if (!unit_T) {
#pragma unroll
      for (int j = 0; j < 8; ++j) zt[j] /= T;                // z / 1 == z exactly: skipped at T = 1
    }
    // running logsumexp, rescaled once per 8 tokens (hardware exponential,
    // relative error ~1e-7)
    float bm = zt[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) bm = fmaxf(bm, zt[j]);
    if (bm > m) { sum *= __expf(m - bm); m = bm; }
#pragma unroll
    for (int j = 0; j < 8; ++j) sum += __expf(zt[j] - m);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t bits = (uint32_t)(w.v[j >> 1] >> (32 * (j & 1)));
      float sc = fmaf(-LN2, gumbel_log2(bits), zt[j]);
      if (vb == eos_vb && j == eos_j) sc = -INFINITY;
      // a thread scans increasing ids, so a strict > keeps the lowest id of a tie
      if (sc > best) { best = sc; best_v = vb * 8 + j; }
    }
    if (a.dump_logits && t < a.dump_steps) {
      float* dst = a.dump_logits + ((int64_t)t * a.n_seq + s) * a.V + vb * 8;
      *reinterpret_cast<float4*>(dst) = z0;
      *reinterpret_cast<float4*>(dst + 4) = z1;
    }
  }
  __shared__ float sb[SAMPLE_THREADS], sm[SAMPLE_THREADS], ss[SAMPLE_THREADS];
  __shared__ int sv[SAMPLE_THREADS];
  sb[tid] = best; sv[tid] = best_v; sm[tid] = m; ss[tid] = sum;
  __syncthreads();
  for (int o = SAMPLE_THREADS / 2; o > 0; o >>= 1) {
    if (tid < o) {
      const float b2 = sb[tid + o]; const int v2 = sv[tid + o];
      if (b2 > sb[tid] || (b2 == sb[tid] && v2 < sv[tid])) { sb[tid] = b2; sv[tid] = v2; }
      const float m1 = sm[tid], m2 = sm[tid + o];
      const float mm = fmaxf(m1, m2);
      ss[tid] = (m1 == -INFINITY ? 0.f : ss[tid] * expf(m1 - mm)) + (m2 == -INFINITY ? 0.f : ss[tid + o] * expf(m2 - mm));
      sm[tid] = mm;
    }
    __syncthreads();
  }
  if (tid == 0) {
    float* p = a.part + ((int64_t)r * a.n_slices + blockIdx.x) * 4;
    p[0] = sb[0];
    p[1] = __int_as_float(sv[0]);
    p[2] = sm[0];
    p[3] = ss[0];
  }
}

// Token of row r from its slices, by the W lanes of a wave (W = 64, or a half of
// 32): lane l combines slices l, l + W, ... in order, then the lanes' results
// are combined (best score, ties to the lowest id; logsumexp by max and
// rescaled sums) and lane 0 decides and writes the outputs.  Every lane of the
// wave calls it; live = false idles through the shuffles.
template <int W>
__device__ __forceinline__ void sample_pick(const SampleArgs& a, int r, int lane, bool live) {
  float best = -INFINITY, m = -INFINITY, sum = 0.f;
  int y = 0x7FFFFFFF;
  for (int k = lane; live && k < a.n_slices; k += W) {
    const float4 p = *reinterpret_cast<const float4*>(a.part + ((int64_t)r * a.n_slices + k) * 4);
    const int v2 = __float_as_int(p.y);
    if (p.x > best || (p.x == best && v2 < y)) { best = p.x; y = v2; }
    const float mm = fmaxf(m, p.z);
    sum = (m == -INFINITY ? 0.f : sum * expf(m - mm)) + (p.z == -INFINITY ? 0.f : p.w * expf(p.z - mm));
    m = mm;
  }
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) {
    const float b2 = __shfl_xor(best, o, 64), m2 = __shfl_xor(m, o, 64), s2 = __shfl_xor(sum, o, 64);
    const int v2 = __shfl_xor(y, o, 64);
    if (b2 > best || (b2 == best && v2 < y)) { best = b2; y = v2; }
    const float mm = fmaxf(m, m2);
    sum = (m == -INFINITY ? 0.f : sum * expf(m - mm)) + (m2 == -INFINITY ? 0.f : s2 * expf(m2 - mm));
    m = mm;
  }
  if (lane != 0 || !live) return;
  const int t = *a.d_t;
  const int s = a.act_seq[r];
  const int lrow = a.logits_by_group ? a.seq_grp[s] : r;
  const float* z = a.logits + (int64_t)lrow * a.V;
  const int L = a.forced_len ? a.forced_len[s] : -1;
  if (L > 0 && t == L - 1) y = a.eos;
  int fed = a.force_tokens ? a.force_tokens[(int64_t)s * a.max_new + t] : y;
  if (fed < 0 || fed >= a.V) { fed = a.eos; a.bad_token[0] = 1; }   // invalid forced id: stop this sequence
  const float lse = m + logf(sum);
  const float lp = z[fed] / a.temperature - lse;
  a.tokens_out[(int64_t)s * a.max_new + t] = y;
  a.logprobs_out[(int64_t)s * a.max_new + t] = lp;
  a.next_tok[r] = fed;
  a.done[r] = (fed == a.eos || t + 1 == a.max_new) ? 1 : 0;
}

__global__ __launch_bounds__(64) void k_sample_pick(SampleArgs a) {
  const int r = blockIdx.x;
  if (r >= *a.d_rows) return;
  sample_pick<64>(a, r, threadIdx.x, true);
}

// ------------------------------------------------------------------ retirement
// One block.  Pass 1 retires finished rows (length, private pages back to the
// free stack); pass 2 compacts the surviving rows in place (stable) and gives
// each survivor whose next position starts a page a fresh page.  PICK: half a
// wave per row first picks the tokens, which saves small batches the pick's
// launch (4.6 us).  The step's state goes to pinned host memory from here, in
// place of a copy per step (4.1 us).
template <bool PICK>
__global__ __launch_bounds__(1024) void k_compact(CompactArgs a, SampleArgs pick) {
  __shared__ int lds[17];
  __shared__ unsigned long long s_ctx;
  __shared__ int s_groups;
  const int tid = threadIdx.x;
  const int M = a.state[0];
  const int t = a.state[8];
  int top = a.state[1];
  if (tid == 0) { s_ctx = 0; s_groups = 0; }
  if constexpr (PICK) sample_pick<32>(pick, tid >> 5, tid & 31, (tid >> 5) < M);
  __syncthreads();   // also orders the picked rows' next_tok and done ahead of their reads
  // pass 1
  int carry = 0;
  for (int base = 0; base < M; base += blockDim.x) {
    const int r = base + tid;
    int f = 0, s = -1;
    bool dn = false;
    if (r < M) {
      s = a.act_seq[r];
      dn = a.done[r] != 0;
      const int p = a.seq_grp[s];
      atomicAdd(&s_ctx, (unsigned long long)a.plen[p]);
      if (r == 0 || a.seq_grp[a.act_seq[r - 1]] != p) atomicAdd(&s_groups, 1);
      if (dn) f = a.seq_npages[s] - a.seq_nshared[s];
    }
    int tot;
    const int off = block_excl_scan(f, lds, &tot) + carry;
    if (dn) {
      a.lengths[s] = t + 1;
      const int32_t* tab = a.page_tab + (int64_t)s * a.max_pages + a.seq_nshared[s];
      for (int i = 0; i < f; ++i) a.free_stack[top + off + i] = tab[i];
      a.seq_npages[s] = a.seq_nshared[s];
    }
    carry += tot;
  }
  top += carry;
  __syncthreads();
  // pass 2
  int kcarry = 0, ncarry = 0;
  bool oom = false;
  for (int base = 0; base < M; base += blockDim.x) {
    const int r = base + tid;
    int s = -1, tok = 0, keep = 0, need = 0;
    if (r < M) {
      s = a.act_seq[r];
      tok = a.act_tok[r];
      keep = a.done[r] == 0;
      need = keep && ((a.plen[a.seq_grp[s]] + t) % a.page_tok == 0);
    }
    __syncthreads();   // every read of this tile precedes any in-place write
    int ktot, ntot;
    const int kidx = block_excl_scan(keep, lds, &ktot) + kcarry;
    const int nidx = block_excl_scan(need, lds, &ntot) + ncarry;
    if (keep) { a.act_seq[kidx] = s; a.act_tok[kidx] = tok; }
    if (need) {
      const int slot = top - 1 - nidx;
      const int np = a.seq_npages[s];
      if (slot >= 0 && np < a.max_pages) {
        a.page_tab[(int64_t)s * a.max_pages + np] = a.free_stack[slot];
        a.seq_npages[s] = np + 1;
      }
    }
    kcarry += ktot;
    ncarry += ntot;
  }
  if (ncarry > top) oom = true;
  // pass 3: row range of every prompt among the kept rows (in sequence
  // order, so each prompt's rows are contiguous)
  const int M2 = oom ? 0 : kcarry;
  for (int p = tid; p < a.P; p += blockDim.x) { a.grp_row0[p] = 0; a.grp_row1[p] = 0; }
  __syncthreads();   // the resets and the compacted act_seq precede the range writes
  for (int r = tid; r < M2; r += blockDim.x) {
    const int p = a.seq_grp[a.act_seq[r]];
    if (r == 0 || a.seq_grp[a.act_seq[r - 1]] != p) a.grp_row0[p] = r;
    if (r == M2 - 1 || a.seq_grp[a.act_seq[r + 1]] != p) a.grp_row1[p] = r + 1;
  }
  if (tid == 0) {
    if (t < a.hist_cap) {
      a.hist_active[t] = M;
      a.hist_groups[t] = s_groups;
      a.hist_ctx[t] = (int64_t)s_ctx;
    }
    if (oom) { a.state[2] = 1; a.state[0] = 0; }
    else { a.state[0] = kcarry; a.state[1] = top - ncarry; }
    a.state[8] = t + 1;   // the next step
    int32_t* slot = a.ring + 8 * (t % a.ring_slots);
    for (int i = 0; i < 8; ++i) slot[i] = a.state[i];
    __threadfence_system();
  }
}

// ------------------------------------------------------------------ fork
// One block.  Sequence s (prompt p, sibling j) gets the prompt's full pages
// by reference (shared) and private copies of the rest: the partial last
// page, or every page when sharing is off.
__global__ __launch_bounds__(1024) void k_fork(ForkArgs a) {
  __shared__ int lds[17];
  const int tid = threadIdx.x;
  int top = a.state[1];
  int carry = 0;
  for (int base = 0; base < a.n_seq; base += blockDim.x) {
    const int s = base + tid;
    int need = 0, p = 0, n_pref = 0, shared = 0;
    if (s < a.n_seq) {
      int lo = 0, hi = a.P - 1;   // last p with grp_off[p] <= s
      while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (a.grp_off[mid] <= s) lo = mid; else hi = mid - 1;
      }
      p = lo;
      const int L = a.plen[p];
      const int n_full = L / a.page_tok;
      n_pref = (L + a.page_tok - 1) / a.page_tok;
      shared = a.share ? n_full : 0;
      need = n_pref - shared;
    }
    int tot;
    const int off = block_excl_scan(need, lds, &tot) + carry;
    if (s < a.n_seq) {
      a.seq_grp[s] = p;
      a.act_seq[s] = s;
      a.seq_npages[s] = n_pref;
      a.seq_nshared[s] = shared;
      const int32_t* ptab = a.page_tab + (int64_t)(a.n_seq + p) * a.max_pages;
      int32_t* stab = a.page_tab + (int64_t)s * a.max_pages;
      for (int i = 0; i < shared; ++i) stab[i] = ptab[i];
      for (int i = 0; i < need; ++i) {
        const int k = off + i;
        const int slot = top - 1 - k;
        const int pg = slot >= 0 ? a.free_stack[slot] : 0;
        stab[shared + i] = pg;
        a.copy_pairs[2 * k] = ptab[shared + i];
        a.copy_pairs[2 * k + 1] = pg;
      }
    }
    carry += tot;
  }
  __syncthreads();
  if (tid == 0) {
    if (carry > top) { a.state[2] = 1; a.state[0] = 0; a.state[3] = 0; }
    else { a.state[1] = top - carry; a.state[3] = carry; }
  }
}

// ------------------------------------------------------------------ set-up
__global__ __launch_bounds__(1024) void k_setup_scan(SetupArgs a) {
  __shared__ int lds[17];
  const int tid = threadIdx.x;
  int c_tok = 0, c_seq = 0, c_pg = 0;
  for (int base = 0; base < a.P; base += blockDim.x) {
    const int p = base + tid;
    const int L = p < a.P ? a.plen[p] : 0;
    const int g = p < a.P ? a.G[p] : 0;
    const int np = (L + a.page_tok - 1) / a.page_tok;
    int t1, t2, t3;
    const int o1 = block_excl_scan(L, lds, &t1) + c_tok;
    const int o2 = block_excl_scan(g, lds, &t2) + c_seq;
    const int o3 = block_excl_scan(np, lds, &t3) + c_pg;
    if (p < a.P) {
      a.prompt_off[p] = o1;
      a.grp_off[p] = o2;
      a.last_rows[p] = o1 + L - 1;
      int32_t* tab = a.page_tab + (int64_t)(a.n_seq + p) * a.max_pages;
      for (int i = 0; i < np; ++i) tab[i] = o3 + i;   // prompt p's pages are consecutive
    }
    c_tok += t1; c_seq += t2; c_pg += t3;
  }
  if (tid == 0) {
    a.prompt_off[a.P] = c_tok;
    a.grp_off[a.P] = c_seq;
    const bool oom = (int64_t)c_pg > a.pool_pages;
    a.state[0] = oom ? 0 : a.n_seq;
    a.state[1] = oom ? 0 : (int)(a.pool_pages - c_pg);
    a.state[2] = oom ? 1 : 0;
    a.state[3] = 0;
    a.state[4] = c_pg;
    a.state[5] = oom ? 0 : c_tok;   // no prefill rows (so no page writes) without room
    a.state[6] = oom ? 0 : a.P;
    a.state[7] = 0;
    a.state[8] = 0;
  }
}

__global__ void k_setup_free(int32_t* free_stack, const int32_t* state, int64_t pool_pages) {
  const int64_t used = state[4];
  const int64_t n = pool_pages - used;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    free_stack[i] = (int32_t)(used + i);
}

__global__ void k_setup_out(int32_t* tokens, float* logprobs, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    if (tokens) tokens[i] = -1;
    logprobs[i] = 0.f;
  }
}

// ------------------------------------------------------------------ advantage
// Small groups leave these kernels bound by the length of their load chain (G,
// then rewards), not by work: segments of SW lanes take a group each, so that
// groups of 16 run four to a wave, and up to a block's width of groups are
// validated and placed by one load and one barrier (group_offsets).  Wider
// sets of groups walk tiles of 1024.

// Advantages of one group of gs members at o0 (0: idle through the shuffles) by
// W neighbouring lanes of a wave (this one sl, all of them mask): mean and
// deviation in fp64.  Every lane of the wave calls it.
template <int W>
__device__ __forceinline__ void advantage_group(const float* __restrict__ rewards, int o0, int gs, int sl,
                                                uint64_t mask, double eps, int ddof, float* __restrict__ adv) {
  const float r0 = gs > 0 ? rewards[o0] : 0.f;
  const float v0 = sl < gs ? rewards[o0 + sl] : 0.f;   // the lane's first member stays in a register
  double sum = 0.0;
  int diff = 0;
  for (int i = sl; i < gs; i += W) {
    const float v = i == sl ? v0 : rewards[o0 + i];
    sum += (double)v;
    diff |= (v != r0);
  }
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  const bool varies = (__ballot(diff) & mask) != 0;
  const double mu = sum / (double)max(gs, 1);
  double sq = 0.0;
  for (int i = sl; i < gs; i += W) {
    const double dv = (double)(i == sl ? v0 : rewards[o0 + i]) - mu;
    sq += dv * dv;
  }
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
  const bool flat = !varies || gs - ddof <= 0;
  const double sigma = flat ? 0.0 : sqrt(sq / (double)(gs - ddof));
  for (int i = sl; i < gs; i += W)
    adv[o0 + i] = flat ? 0.f : (float)(((double)(i == sl ? v0 : rewards[o0 + i]) - mu) / (sigma + eps));
}

// Groups k = seg, seg + nseg, ... < ng whose offsets are offs[k] .. offs[k + 1],
// a segment of SW lanes each: f(width, k, o0, gs, sl, mask) is called by the
// whole wave, gs = 0 where a segment has no group.  The width follows the
// groups' average; those of more than four rounds of a segment are left to the
// whole wave, so that a large group among small ones is not walked by few lanes
// (1024 among 63 of 4 members, advantage: 15.0 -> 10.7 us).
template <int SW, typename F>
__device__ __forceinline__ void group_tile(const int* offs, int ng, F&& f) {
  const int tid = threadIdx.x, lane = tid & 63, sl = tid % SW, nseg = blockDim.x / SW;
  const uint64_t mask = SW == 64 ? ~0ull : ((1ull << SW) - 1) << (lane / SW * SW);
  constexpr int WIDE = 4 * SW;
  bool any_wide = false;
  for (int k0 = 0; k0 < ng; k0 += nseg) {
    const int k = k0 + tid / SW;
    const bool live = k < ng;   // whole segments; the others idle through the shuffles
    const int o0 = live ? offs[k] : 0, gs = live ? offs[k + 1] - o0 : 0;
    const bool wide = SW < 64 && gs > WIDE;
    any_wide |= wide;
    f(std::integral_constant<int, SW>(), k, o0, wide ? 0 : gs, sl, mask);
  }
  if (SW == 64 || !__any(any_wide)) return;
  for (int k0 = 0; k0 < ng; k0 += nseg) {
    const int k = k0 + tid / SW;
    const bool wide = sl == 0 && k < ng && offs[k + 1] - offs[k] > WIDE;
    for (uint64_t todo = __ballot(wide); todo; todo &= todo - 1) {
      const int kw = __shfl(k, __ffsll((unsigned long long)todo) - 1, 64), o0 = offs[kw];
      f(std::integral_constant<int, 64>(), kw, o0, offs[kw + 1] - o0, lane, ~0ull);
    }
  }
}

template <int SW>
__device__ __forceinline__ void advantage_tile(const float* __restrict__ rewards, const int* offs, int ng, double eps,
                                               int ddof, float* __restrict__ adv) {
  group_tile<SW>(offs, ng, [&](auto w, int, int o0, int gs, int sl, uint64_t mask) {
    advantage_group<decltype(w)::value>(rewards, o0, gs, sl, mask, eps, ddof, adv);
  });
}

template <int SW>
__global__ __launch_bounds__(1024) void k_group_advantage(const float* __restrict__ rewards,
                                                          const int32_t* __restrict__ G, int P, int N, double eps,
                                                          int ddof, float* __restrict__ adv) {
  __shared__ int lds[17];
  __shared__ int offs[1025];
  const int tid = threadIdx.x;
  const bool one = P <= (int)blockDim.x;
  int g1 = 0, o1 = 0;
  const bool ok = one ? group_offsets(G, P, N, g1, o1) : groups_valid(G, P, N);
  if (!ok) {
    for (int i = tid; i < N; i += blockDim.x) adv[i] = __int_as_float(0x7FC00000);
    return;
  }
  if (one) {
    if (tid < P) offs[tid] = o1;
    if (tid == 0) offs[P] = N;
    __syncthreads();
    advantage_tile<SW>(rewards, offs, P, eps, ddof, adv);
    return;
  }
  int carry = 0;
  for (int base = 0; base < P; base += blockDim.x) {
    const int p = base + tid;
    const int g = p < P ? G[p] : 0;
    int t;
    const int o = block_excl_scan(g, lds, &t) + carry;
    offs[tid] = o;
    if (tid == (int)blockDim.x - 1) offs[blockDim.x] = o + g;
    __syncthreads();
    advantage_tile<SW>(rewards, offs, min((int)blockDim.x, P - base), eps, ddof, adv);
    carry += t;
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_gumbel_noise(uint32_t first, int64_t n, float* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gumbel_noise, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, first, n, out);
  return hipGetLastError();
}

hipError_t launch_sample(const SampleArgs& a, int rows_ub, bool pick, hipStream_t st) {
  if (rows_ub <= 0) return hipSuccess;
  if (a.n_slices < 1 || a.V % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_sample_slice, dim3(a.n_slices, rows_ub), dim3(SAMPLE_THREADS), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !pick) return e;
  hipLaunchKernelGGL(k_sample_pick, dim3(rows_ub), dim3(64), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_compact(const CompactArgs& a, const SampleArgs* pick, hipStream_t st) {
  if (!a.ring || a.ring_slots < 1) return hipErrorInvalidValue;
  if (pick && pick->n_slices > COMPACT_PICK_SLICES) return hipErrorInvalidValue;
  if (pick) hipLaunchKernelGGL(k_compact<true>, dim3(1), dim3(1024), 0, st, a, *pick);
  else hipLaunchKernelGGL(k_compact<false>, dim3(1), dim3(1024), 0, st, a, SampleArgs{});
  return hipGetLastError();
}

hipError_t launch_fork(const ForkArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_fork, dim3(1), dim3(1024), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_setup(const SetupArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_setup_scan, dim3(1), dim3(1024), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_setup_free, dim3(1024), dim3(256), 0, st, a.free_stack, a.state, a.pool_pages);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t n = (int64_t)a.n_seq * a.max_new;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_setup_out, dim3((unsigned)blocks), dim3(256), 0, st, a.tokens_out, a.logprobs_out, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------ group length statistics
// One block of four waves per group: the group's offset is the sum of the sizes
// before it; its lengths are ranked in LDS (rank = smaller values plus equal
// values earlier in the group) and placed in sorted order.  The first wave
// alone, without a barrier, takes a group of at most 64; the average says
// nothing about a large group among small ones (1024 among 63 of 4 members, us a
// launch: 463 on the one wave that the average asks for, 107 on four).
__global__ __launch_bounds__(256) void k_group_stats(const int32_t* __restrict__ lengths, const int32_t* __restrict__ G,
                                                     int P, int N, double tau, float* __restrict__ stats) {
  constexpr int GMAX = 1024;
  __shared__ int s_len[GMAX], s_sorted[GMAX];
  __shared__ long long s_off[4];
  const int64_t pb = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (pb >= P) return;
  const int p = (int)pb, tid = threadIdx.x, lane = tid & 63;
  const int g = G[p];
  const bool small = g <= 64;
  long long off = 0;   // integer sum: order-independent, exact for int32 sizes
  if (P <= 256) {      // each wave sums all sizes itself
    if (small && tid >= 64) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) off += lane + 64 * u < p ? (long long)G[lane + 64 * u] : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) off += __shfl_xor(off, o, 64);
  } else {
    long long part = 0;
    for (int i = tid; i < p; i += 256) part += (long long)G[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
    if (lane == 0) s_off[tid >> 6] = part;
    __syncthreads();
    off = (s_off[0] + s_off[1]) + (s_off[2] + s_off[3]);
    if (small && tid >= 64) return;
  }
  float* out = stats + 4 * (int64_t)p;
  if (g < 1 || g > GMAX || off < 0 || off + g > N) {
    if (tid < 4) out[tid] = NAN;
    return;
  }
  // what the group's threads (nt of them) wrote to LDS is seen by all of them
  auto sync = [&]() {
    if (small) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    } else {
      __syncthreads();
    }
  };
  const int nt = small ? 64 : 256;
  for (int i = tid; i < g; i += nt) s_len[i] = lengths[off + i];
  sync();
  for (int i = tid; i < g; i += nt) {
    const int v = s_len[i];
    int rank = 0;
    if (small) {
#pragma unroll 4
      for (int j = 0; j < g; ++j) {
        const int u = s_len[j];
        rank += (u < v) || (u == v && j < i);
      }
    } else {
      for (int j = 0; j < g; ++j) {
        const int u = s_len[j];
        rank += (u < v) || (u == v && j < i);
      }
    }
    s_sorted[rank] = v;
  }
  sync();
  if (tid == 0) {
    const int lmax = s_sorted[g - 1];
    const double med = (g & 1) ? (double)s_sorted[g / 2] : ((double)s_sorted[g / 2 - 1] + (double)s_sorted[g / 2]) / 2.0;
    if (!(med > 0.0)) {
      out[0] = out[1] = out[2] = out[3] = NAN;
      return;
    }
    const double R = (double)lmax / med;
    out[0] = (float)lmax;
    out[1] = (float)med;
    out[2] = (float)R;
    out[3] = R > tau ? 1.f : 0.f;
  }
}

hipError_t launch_group_stats(const int32_t* lengths, const int32_t* G, int P, int N, double tau, float* stats,
                              hipStream_t st) {
  if (P < 1) return hipSuccess;
  // a launch holds fewer than 2^32 threads in a dimension: past 2^20 groups in rows of blocks
  const int gx = std::min(P, 1 << 20);
  hipLaunchKernelGGL(k_group_stats, dim3(gx, (unsigned)(((int64_t)P + gx - 1) / gx)), dim3(256), 0, st, lengths, G, P, N,
                     tau, stats);
  return hipGetLastError();
}

// ------------------------------------------------------------------ zero-variance filter
// One block.  Validates G as the advantage does; then a segment of SW lanes
// per group, or a lane where the segments would take several rounds, compares
// its rewards with the first one (exact fp32 equality) and a scan compacts the
// ids of the groups that vary.  n_kept[0] = number of kept
// groups, or -1 when G is invalid (nothing else written).
template <int SW>
__device__ __forceinline__ void filter_tile(const float* __restrict__ rewards, const int* offs, int ng, int* var) {
  group_tile<SW>(offs, ng, [&](auto w, int k, int o0, int gs, int sl, uint64_t mask) {
    const float r0 = gs > 0 ? rewards[o0] : 0.f;
    int diff = 0;
    for (int i = sl; i < gs; i += decltype(w)::value) diff |= i > 0 && rewards[o0 + i] != r0;
    const bool varies = (__ballot(diff) & mask) != 0;
    if (gs > 0 && sl == 0) var[k] = varies;   // every valid group has a member
  });
}

// The same for a lane's own group (g members at o; 0: none).  It ends at the
// first member that differs; a group alike through its first 128 is left to the
// whole wave.  Every lane of the wave calls it.
__device__ __forceinline__ int filter_lane(const float* __restrict__ rewards, int o, int g) {
  constexpr int LANE_MAX = 128;
  const int lane = threadIdx.x & 63;
  const float r0 = g > 0 ? rewards[o] : 0.f;
  int diff = 0;
  for (int i = 1; i < min(g, LANE_MAX) && !diff; i += 4) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = rewards[o + min(i + u, g - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) diff |= v[u] != r0;
  }
  for (uint64_t todo = __ballot(!diff && g > LANE_MAX); todo; todo &= todo - 1) {
    const int src = __ffsll((unsigned long long)todo) - 1;
    const int wo = __shfl(o, src, 64), wg = __shfl(g, src, 64);
    const float w0 = __shfl(r0, src, 64);
    int d = 0;
    for (int i = LANE_MAX + lane; i < wg; i += 64) d |= rewards[wo + i] != w0;
    if (__any(d) && lane == src) diff = 1;
  }
  return diff;
}

template <int SW>
__global__ __launch_bounds__(1024) void k_group_filter(const float* __restrict__ rewards, const int32_t* __restrict__ G,
                                                      int P, int N, int32_t* __restrict__ keep,
                                                      int32_t* __restrict__ kept_ids, int32_t* __restrict__ n_kept) {
  __shared__ int lds[17];
  __shared__ int offs[1025], var[1024];
  const int tid = threadIdx.x;
  const bool one = P <= (int)blockDim.x;
  int g1 = 0, o1 = 0;
  const bool ok = one ? group_offsets(G, P, N, g1, o1) : groups_valid(G, P, N);
  if (!ok) {
    if (tid == 0) n_kept[0] = -1;
    return;
  }
  int carry = 0, kcarry = 0;
  for (int base = 0; base < P; base += blockDim.x) {
    const int p = base + tid;
    if (one) {
      if (tid < P) offs[tid] = o1;
      if (tid == 0) offs[P] = N;
    } else {
      const int g = p < P ? G[p] : 0;
      int t;
      const int o = block_excl_scan(g, lds, &t) + carry;
      offs[tid] = o;
      if (tid == (int)blockDim.x - 1) offs[blockDim.x] = o + g;
      carry += t;
    }
    __syncthreads();
    filter_tile<SW>(rewards, offs, min((int)blockDim.x, P - base), var);
    __syncthreads();
    const int varies = p < P ? var[tid] : 0;
    int kt;
    const int k = block_excl_scan(varies, lds, &kt) + kcarry;
    if (p < P) keep[p] = varies;
    if (varies) kept_ids[k] = p;
    kcarry += kt;
    __syncthreads();
  }
  if (tid == 0) n_kept[0] = kcarry;
}

__global__ __launch_bounds__(1024) void k_group_filter_lanes(const float* __restrict__ rewards,
                                                            const int32_t* __restrict__ G, int P, int N,
                                                            int32_t* __restrict__ keep,
                                                            int32_t* __restrict__ kept_ids,
                                                            int32_t* __restrict__ n_kept) {
  __shared__ int lds[17];
  const int tid = threadIdx.x;
  const bool one = P <= (int)blockDim.x;
  int g = 0, o = 0;
  const bool ok = one ? group_offsets(G, P, N, g, o) : groups_valid(G, P, N);
  if (!ok) {
    if (tid == 0) n_kept[0] = -1;
    return;
  }
  int carry = 0, kcarry = 0;
  for (int base = 0; base < P; base += blockDim.x) {
    const int p = base + tid;
    if (!one) {
      int t;
      g = p < P ? G[p] : 0;
      o = block_excl_scan(g, lds, &t) + carry;
      carry += t;
    }
    const int varies = filter_lane(rewards, o, g);
    int kt;
    const int k = block_excl_scan(varies, lds, &kt) + kcarry;
    if (p < P) keep[p] = varies;
    if (varies) kept_ids[k] = p;
    kcarry += kt;
  }
  if (tid == 0) n_kept[0] = kcarry;
}

namespace {
// Lanes per group (16 to 64, at least the average size) and block threads (a
// segment per group up to 1024 threads, at least P so that one load covers G).
int group_lanes(int P, int N) { return N / P <= 16 ? 16 : N / P <= 32 ? 32 : 64; }
int group_threads(int P, int lanes) {
  const int64_t t = (int64_t)P * lanes;
  return (int)((t < 64 ? 64 : t > 1024 ? 1024 : t) + 63) / 64 * 64;
}
}  // namespace

#define RG_GROUP_LAUNCH(K, ...)                                                                               \
  do {                                                                                                        \
    const dim3 nt(group_threads(P, lanes));                                                                   \
    if (lanes == 16) hipLaunchKernelGGL(K<16>, dim3(1), nt, 0, st, __VA_ARGS__);                              \
    else if (lanes == 32) hipLaunchKernelGGL(K<32>, dim3(1), nt, 0, st, __VA_ARGS__);                         \
    else hipLaunchKernelGGL(K<64>, dim3(1), nt, 0, st, __VA_ARGS__);                                          \
  } while (0)

// A lane per group, which stops early, once the segments would take more than
// one round of a 1024-thread block (512 groups of 16: 7.0 -> 4.5 us, 4096 of 4:
// 35 -> 15).
hipError_t launch_group_filter(const float* rewards, const int32_t* G, int P, int N, int32_t* keep, int32_t* kept_ids,
                               int32_t* n_kept, hipStream_t st) {
  const int lanes = group_lanes(P, N);
  if ((int64_t)P * lanes > 1024)
    hipLaunchKernelGGL(k_group_filter_lanes, dim3(1), dim3(group_threads(P, 1)), 0, st, rewards, G, P, N, keep,
                       kept_ids, n_kept);
  else
    RG_GROUP_LAUNCH(k_group_filter, rewards, G, P, N, keep, kept_ids, n_kept);
  return hipGetLastError();
}

hipError_t launch_group_advantage(const float* rewards, const int32_t* G, int P, int N, float eps, int ddof,
                                  float* adv, hipStream_t st) {
  const int lanes = group_lanes(P, N);
  RG_GROUP_LAUNCH(k_group_advantage, rewards, G, P, N, (double)eps, ddof, adv);
  return hipGetLastError();
}
#undef RG_GROUP_LAUNCH
