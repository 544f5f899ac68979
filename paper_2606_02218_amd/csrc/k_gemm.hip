// Matrix products of the decoder, y = x W^T with activations [rows, K] and
// weights W [N, K] (both K-contiguous), each with a fused epilogue:
//   STORE     C[r][n] = y                          (lm head logits)
//   RESIDUAL  x[r][n] += y                         (O and down projections),
//             and for the next RMSNorm the operand x * gain and partial sums of
//             x^2 per row
//   SWIGLU    act[r][f] = silu(gate) * up          (gate/up projection; packed
//             columns come as [16 gate | 16 up] per 32)
//   LOGPROB   the lm head of scored rows: no logits, but each row's logsumexp
//             over the tile's columns and the logit of the token it predicts
//   QKV       RoPE on the query and key heads; q -> fp32 buffer, k and v ->
//             the row's KV page (keys as [slot][dim], values as [dim][slot]).
//             Within each head the packed weight rows come in 16-row tiles
//             ordered (dims 0-15, dims h/2..h/2+15, dims 16-31, ...) so that
//             a rotated pair (d, d + h/2) lies in adjacent column tiles.
//
// RMSNorm has no launch of its own: the producer of x leaves x * gain as the
// next operand and, per row and column tile, the sum of x^2; the consumer's
// products are scaled by the row's 1 / rms in its epilogue (the factor is the
// same for the whole row, and the hi/lo split is relative, so the precision is
// that of splitting the normalised value).
//
// bf16 models: LDS-tiled gfx950 MFMA (v_mfma_f32_16x16x32_bf16).  A block
// owns a BM x BN output tile and walks its K range in steps of 64.  The
// activation comes as hi/lo bf16 planes and every fragment takes two MFMAs
// (W*hi + W*lo) into one fp32 accumulator; each wave owns a WM x WN grid of 16
// x 16 MFMA tiles.  Two kernels: k_gemm_tiled (few rows: every thread fetches
// 16-byte pieces of the next A and W tiles into registers while the waves
// multiply the current tiles out of LDS) and k_gemm_dma (128-row tiles, loads
// straight into a second LDS buffer).
//
// Split over K: the grid's z dimension splits K and every split writes its
// fp32 partial; k_split_epilogue then sums the partials in split order (one
// block per row and 128 columns) and runs the epilogue.  Without a split the
// epilogue runs straight from the accumulators.
//
// MFMA 16x16x32 lane layout: lane l supplies row (l % 16), k-slice
// 8*(l / 16) .. +7 of A and column (l % 16), the same k-slice of B; it
// receives C rows 4*(l / 16) .. +3 of column (l % 16).
#include <algorithm>

#include "rg_device.h"
#include "rg_kernels.h"

namespace {

constexpr int BK = 64;                 // K step
constexpr int LDS_PAD = 16;            // bf16 elements of padding per LDS row (rows 160 B apart: no bank conflicts)

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t lds_frag(const bf16_t* p) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(p));
}

// 1 / rms of a block's BM rows from the ep.ssq_n partial sums of squares of each
// (NULL ep.ssq_in: the operand is already normalised, factor 1).  NT / BM
// threads share a row; load() issues the first eight partials of a thread,
// finish() adds them up once the K loop is over.
template <int BM, int NT>
struct RowScale {
  static constexpr int TPR = NT / BM, U = 8;
  static_assert(NT % BM == 0 && TPR <= 64 && (TPR & (TPR - 1)) == 0, "threads per row");
  float v[U];
  __device__ __forceinline__ void load(const GemmEpi& ep, int m0, int rows_cap, int tid) {
    const float* p = ep.ssq_in + (int64_t)min(m0 + tid / TPR, rows_cap - 1) * ep.ssq_ld;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = tid % TPR + u * TPR;
      v[u] = ep.ssq_in && k < ep.ssq_n ? p[k] : 0.f;
    }
  }
  __device__ __forceinline__ void finish(const GemmEpi& ep, int m0, int rows_cap, int tid, float* s_inv) {
    float s = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) s += v[u];
    if (ep.ssq_in) {
      const float* p = ep.ssq_in + (int64_t)min(m0 + tid / TPR, rows_cap - 1) * ep.ssq_ld;
      for (int k = tid % TPR + U * TPR; k < ep.ssq_n; k += TPR) s += p[k];
    }
#pragma unroll
    for (int o = TPR / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (tid % TPR == 0) s_inv[tid / TPR] = ep.ssq_in ? 1.0f / sqrtf(s / (float)ep.norm_dim + ep.norm_eps) : 1.f;
    __syncthreads();
  }
};

// The same factor for row r, the same for every lane of a wave.
__device__ __forceinline__ float wave_row_scale(const GemmEpi& ep, int r, int lane) {
  if (!ep.ssq_in) return 1.f;
  const float* p = ep.ssq_in + (int64_t)r * ep.ssq_ld;
  float s = 0.f;
  for (int k = lane; k < ep.ssq_n; k += 64) s += p[k];
  return 1.0f / sqrtf(wave_sum(s) / (float)ep.norm_dim + ep.norm_eps);
}

// Sum of the split partials of element (r, c), in split order.  The loads
// of a batch of 16 splits are all issued before its first add.
__device__ __forceinline__ float split_sum(const GemmEpi& ep, int S, int64_t off) {
  constexpr int BATCH = 16;
  const float* p = ep.part + off;
  const int64_t st = ep.part_stride;
  float acc = 0.f;
  for (int s0 = 0; s0 < S; s0 += BATCH) {
    float v[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) v[j] = s0 + j < S ? p[(s0 + j) * st] : 0.f;
#pragma unroll
    for (int j = 0; j < BATCH; ++j) acc += v[j];
  }
  return acc;
}

// QKV epilogue of row r of an fp32 model for packed column c (a lower-half
// tile column: bit 4 of c is 0) holding dim d of its head, and c + 16 holding
// dim d + half.
__device__ __forceinline__ void qkv_store_f32(const GemmEpi& ep, int r, int c, float a, float b) {
  const int hd = ep.hd, half = hd / 2;
  const int head = c / hd, p = c % hd;
  const int d = (p >> 5) * 16 + (p & 15);
  const int pos = ep.row_pos[r];
  float* pool = (float*)ep.kv_pool;
  if (head >= ep.n_q + ep.n_kv) {                     // value head: no rotation, V^T layout
    const int kvh = head - ep.n_q - ep.n_kv;
    const int page = ep.page_tab[(int64_t)ep.row_tab[r] * ep.tab_stride + pos / 16];
    float* vb = pool + (int64_t)page * ep.geom.page_stride + (int64_t)ep.layer * ep.geom.layer_stride +
                ((int64_t)ep.n_kv + kvh) * 16 * hd;
    vb[kv_v_off(pos & 15, d, hd)] = a;
    vb[kv_v_off(pos & 15, d + half, hd)] = b;
    return;
  }
  const float co = ep.rope_cos[(int64_t)pos * half + d], si = ep.rope_sin[(int64_t)pos * half + d];
  const float ra = a * co - b * si, rb = b * co + a * si;
  if (head < ep.n_q) {
    float* qo = ep.q_out + ((int64_t)r * ep.n_q + head) * hd;
    qo[d] = ra;
    qo[d + half] = rb;
  } else {
    const int kvh = head - ep.n_q;
    const int page = ep.page_tab[(int64_t)ep.row_tab[r] * ep.tab_stride + pos / 16];
    float* kp = pool + (int64_t)page * ep.geom.page_stride + (int64_t)ep.layer * ep.geom.layer_stride +
                (int64_t)kvh * 16 * hd;
    kp[kv_k_off(pos & 15, d)] = ra;
    kp[kv_k_off(pos & 15, d + half)] = rb;
  }
}

// QKV epilogue straight from the accumulators of one wave (rows
// m0 + (wm*WM + i)*16 + 4*(lane/16) + e, column tiles wn*WN + j).  One row
// block i at a time, every load it needs (row position, KV page, the RoPE
// cos/sin of each rotated pair) is issued before the first store: through
// restrict-qualified pointers the loads of a block do not wait on the stores
// of the previous one, so the tile pays a few load latencies instead of one
// per element.
template <int WM, int WN>
__device__ __forceinline__ void qkv_tile_store(const f32x4_t (&acc)[WM][WN], const GemmEpi& ep, int m0, int n0, int M,
                                               int N, int wm, int wn, int lane,
                                               const int32_t* __restrict__ row_pos,
                                               const int32_t* __restrict__ row_tab,
                                               const int32_t* __restrict__ page_tab,
                                               const float* __restrict__ rcos, const float* __restrict__ rsin,
                                               float* __restrict__ q_out, bf16_t* __restrict__ pool) {
  const int lr = lane & 15;
  const int hd = ep.hd, half = hd / 2, n_rot = ep.n_q + ep.n_kv;
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int rb = m0 + (wm * WM + i) * 16 + (lane >> 4) * 4;
    int pos[4];
    int64_t kvb[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = min(rb + e, M - 1);
      pos[e] = row_pos[r];
      const int page = page_tab[(int64_t)row_tab[r] * ep.tab_stride + pos[e] / 16];
      kvb[e] = (int64_t)page * ep.geom.page_stride + (int64_t)ep.layer * ep.geom.layer_stride;
    }
    float co[WN / 2][4], si[WN / 2][4];
#pragma unroll
    for (int j = 0; j < WN; j += 2) {
      const int c = min(n0 + (wn * WN + j) * 16 + lr, N - 1);
      const int p = c % hd, d = (p >> 5) * 16 + (p & 15);
      const bool rot = c / hd < n_rot;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        co[j / 2][e] = rot ? rcos[(int64_t)pos[e] * half + d] : 1.f;
        si[j / 2][e] = rot ? rsin[(int64_t)pos[e] * half + d] : 0.f;
      }
    }
#pragma unroll
    for (int j = 0; j < WN; j += 2) {
      const int c = n0 + (wn * WN + j) * 16 + lr;   // lower tile's column
      if (c >= N) continue;
      const int head = c / hd, p = c % hd, d = (p >> 5) * 16 + (p & 15);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (rb + e >= M) continue;
        const float a = acc[i][j][e], b = acc[i][j + 1][e];
        const int slot = pos[e] & 15;
        if (head >= n_rot) {                               // value head: V^T layout, no rotation
          bf16_t* vb = pool + kvb[e] + ((int64_t)ep.n_kv + head - n_rot) * 16 * hd;
          vb[kv_v_off(slot, d, hd)] = f32_to_bf16(a);
          vb[kv_v_off(slot, d + half, hd)] = f32_to_bf16(b);
          continue;
        }
        const float ra = a * co[j / 2][e] - b * si[j / 2][e], rr = b * co[j / 2][e] + a * si[j / 2][e];
        if (head < ep.n_q) {
          float* qo = q_out + ((int64_t)(rb + e) * ep.n_q + head) * hd;
          qo[d] = ra;
          qo[d + half] = rr;
        } else {
          bf16_t* kp = pool + kvb[e] + (int64_t)(head - ep.n_q) * 16 * hd;
          kp[kv_k_off(slot, d)] = f32_to_bf16(ra);
          kp[kv_k_off(slot, d + half)] = f32_to_bf16(rr);
        }
      }
    }
  }
}

// Epilogues whose operand may be an unnormalised x * gain.
template <int EPI>
constexpr bool kScaled = EPI == GEMM_EPI_STORE || EPI == GEMM_EPI_SWIGLU || EPI == GEMM_EPI_QKV || EPI == GEMM_EPI_LOGPROB;

template <int WM, int WN>
__device__ __forceinline__ void scale_rows(f32x4_t (&acc)[WM][WN], const float* s_inv, int wm, int lane) {
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const f32x4_t f = *reinterpret_cast<const f32x4_t*>(s_inv + (wm * WM + i) * 16 + (lane >> 4) * 4);
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] *= f;
  }
}

// RESIDUAL epilogue of one wave.  The four rows of a block of accumulators are
// loaded at once, and the next block's before this one's stores (which the
// compiler may not move them across): read-modify-write one element after the
// other paid a load latency per element, about as long as the tile's K loop at
// K = 1536.
template <int WM, int WN, int WAVES_N>
__device__ __forceinline__ void residual_tile(const f32x4_t (&acc)[WM][WN], const GemmEpi& ep, bool norm, int m0,
                                              int n0, int M, int N, int wm, int wn, int lane,
                                              float* __restrict__ x, const float* __restrict__ gain,
                                              bf16_t* __restrict__ act, float* s_ssq) {
  const int lr = lane & 15;
  int col[WN];
  float g[WN];
#pragma unroll
  for (int j = 0; j < WN; ++j) {
    const int c = n0 + (wn * WN + j) * 16 + lr;
    col[j] = min(c, N - 1);
    g[j] = norm ? gain[col[j]] : 0.f;
  }
  float xv[2][4][WN];
  auto fetch = [&](int i) {
    const int rl = (wm * WM + i) * 16 + (lane >> 4) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int j = 0; j < WN; ++j) xv[i & 1][e][j] = x[(int64_t)min(m0 + rl + e, M - 1) * ep.ldx + col[j]];
  };
  fetch(0);
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int rl = (wm * WM + i) * 16 + (lane >> 4) * 4;
    if (i + 1 < WM) fetch(i + 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = m0 + rl + e;
      float ss = 0.f;
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const bool on = r < M && n0 + (wn * WN + j) * 16 + lr < N;
        const float v = xv[i & 1][e][j] + acc[i][j][e];
        if (!on) continue;
        ss = fmaf(v, v, ss);
        x[(int64_t)r * ep.ldx + col[j]] = v;
        if (norm) {
          const float a = v * g[j];
          const bf16_t h = f32_to_bf16(a);
          bf16_t* o = act + (int64_t)r * N + col[j];
          o[0] = h;
          o[ep.norm_out.plane] = f32_to_bf16(a - bf16_to_f32(h));
        }
      }
      if (norm) {
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
        if (lr == 0) s_ssq[(rl + e) * WAVES_N + wn] = ss;
      }
    }
  }
}

// Epilogue of one wave straight from its accumulators: rows m0 + (wm*WM + i)*16
// + 4*(lane/16) + e, columns n0 + (wn*WN + j)*16 + lane%16; only rows below M
// and columns below N are stored.
// Every thread of the block calls it; s_ssq holds BM x WAVES_N floats.
template <int EPI, int BM, int WM, int WN, int WAVES_N>
__device__ __forceinline__ void acc_epilogue(const f32x4_t (&acc)[WM][WN], const GemmEpi& ep, int tz, int tx, int m0,
                                             int n0, int M, int N, int wm, int wn, int tid, float* s_ssq) {
  const int lane = tid & 63, lr = lane & 15;
  if constexpr (EPI == GEMM_EPI_PARTIAL) {
    float* pp = ep.part + tz * ep.part_stride;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int col = n0 + (wn * WN + j) * 16 + lr;
        if (col >= N) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = m0 + (wm * WM + i) * 16 + (lane >> 4) * 4 + e;
          if (r < M) pp[(int64_t)r * N + col] = acc[i][j][e];
        }
      }
  } else if constexpr (EPI == GEMM_EPI_QKV) {
    qkv_tile_store<WM, WN>(acc, ep, m0, n0, M, N, wm, wn, lane, ep.row_pos, ep.row_tab, ep.page_tab, ep.rope_cos,
                           ep.rope_sin, ep.q_out, (bf16_t*)ep.kv_pool);
  } else if constexpr (EPI == GEMM_EPI_LOGPROB) {
    // one (max, sum of exp(z/T - max)) per row and wave column, over the wave's
    // columns below N: a lane folds its WN columns, the 16 lanes of a row the
    // rest.  Past N the logit counts as -inf.
    // expf, as where the logits are written: 8.4e-8 relative at most over [-87,
    // 0]; __expf, which rounds x log2(e) first, is off by 5e-7 from -8 and 1e-6
    // from -20 (it takes 3 % off the four-layer 1.5B recompute).
    const float T = ep.temperature;
    const bool unit_T = T == 1.0f;               // z / 1 == z exactly
    const int part = (n0 / (16 * WN)) + wn;      // this wave's column range
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = m0 + (wm * WM + i) * 16 + (lane >> 4) * 4 + e;
        const int tgt = r < M ? ep.row_tgt[r] : -1;
        float z[WN], m = -INFINITY;
#pragma unroll
        for (int j = 0; j < WN; ++j) {
          const int col = n0 + (wn * WN + j) * 16 + lr;
          z[j] = col < N ? (unit_T ? acc[i][j][e] : acc[i][j][e] / T) : -INFINITY;
          if (col == tgt) ep.tgt_z[r] = z[j];    // one lane of the launch per row
          m = fmaxf(m, z[j]);
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < WN; ++j) s += z[j] == -INFINITY ? 0.f : z[j] == m ? 1.f : expf(z[j] - m);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lr == 0 && r < M) ep.lse_part[(int64_t)r * ep.lse_ld + part] = float2{m, s};
      }
  } else if constexpr (EPI == GEMM_EPI_SWIGLU) {
    // tiles 2m and 2m+1 of a wave pair up: (gate, up)
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; j += 2) {
        const int c = n0 + (wn * WN + j) * 16 + lr;   // lower tile's column
        if (c >= N) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = m0 + (wm * WM + i) * 16 + (lane >> 4) * 4 + e;
          if (r >= M) continue;
          const float a = acc[i][j][e], b = acc[i][j + 1][e];
          act_store<1>(ep.act, (int64_t)r * ep.act_ld + (c >> 5) * 16 + lr, a / (1.0f + expf(-a)) * b);
        }
      }
  } else if constexpr (EPI == GEMM_EPI_RESIDUAL) {
    const bool norm = ep.norm_g != nullptr;
    residual_tile<WM, WN, WAVES_N>(acc, ep, norm, m0, n0, M, N, wm, wn, lane, ep.x, ep.norm_g,
                                   (bf16_t*)ep.norm_out.base, s_ssq);
    if (norm) {
      __syncthreads();
      if (tid < BM && m0 + tid < M) {
        float s = s_ssq[tid * WAVES_N];
#pragma unroll
        for (int w = 1; w < WAVES_N; ++w) s += s_ssq[tid * WAVES_N + w];
        ep.ssq_out[(int64_t)(m0 + tid) * ep.ssq_ld + tx] = s;
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int col = n0 + (wn * WN + j) * 16 + lr;
        if (col >= N) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = m0 + (wm * WM + i) * 16 + (lane >> 4) * 4 + e;
          if (r < M) ep.C[(int64_t)r * ep.ldc + col] = acc[i][j][e];
        }
      }
  }
}

// A 16-byte piece of W.  NT: a non-temporal load, for weights that no other
// block of the launch reads (one row tile): streamed through without
// claiming cache space, which measured 6.5-6.7 TB/s against 5.9-6.1 TB/s
// for plain loads in a pure streaming read of 8 GiB.
__host__ __device__ __forceinline__ int k_split_count(int K, int k_per_split) { return (K + k_per_split - 1) / k_per_split; }

template <bool NT>
__device__ __forceinline__ u32x4_t load_w(const bf16_t* p) {
  if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  else return *reinterpret_cast<const u32x4_t*>(p);
}

template <int BM, int BN, int WM, int WN, int EPI, bool NTW>
__global__ __launch_bounds__((BM / (16 * WM)) * (BN / (16 * WN)) * 64) void k_gemm_tiled(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, const int* __restrict__ d_rows, int64_t a_plane,
    int lda, int ldw, int rows_cap, int N, int K, int k_per_split, GemmEpi ep) {
  // The arguments the first loads need come first (14 dwords, which the
  // build preloads into scalar registers at dispatch).  The row count is
  // read first but waited for only after the first K step's loads are
  // issued: those clamp A rows to the launch's row bound rows_cap (>= the
  // count; the activation buffer holds that many rows), so they do not
  // depend on it.  Rows past the count are multiplied, never stored.
  const int rows_now = *d_rows;
  constexpr int WAVES_M = BM / (16 * WM), WAVES_N = BN / (16 * WN);
  constexpr int NT = WAVES_M * WAVES_N * 64;
  constexpr int LROW = BK + LDS_PAD;                // LDS row stride (elements)
  constexpr int A_PIECES = BM * (BK / 8);          // 16-byte pieces per A plane tile
  constexpr int W_PIECES = BN * (BK / 8);
  static_assert((2 * A_PIECES) % NT == 0 && W_PIECES % NT == 0, "tile pieces must split evenly over threads");
  static_assert((EPI != GEMM_EPI_SWIGLU && EPI != GEMM_EPI_QKV) || WN % 2 == 0, "pairs of adjacent column tiles");
  constexpr int A_PER_T = 2 * A_PIECES / NT;
  constexpr int W_PER_T = W_PIECES / NT;
  __shared__ __attribute__((aligned(16))) bf16_t sA[2][BM * LROW];
  __shared__ __attribute__((aligned(16))) bf16_t sW[BN * LROW];

  const int tx = blockIdx.x, ty = blockIdx.y, tz = blockIdx.z;
  const int m0 = ty * BM;   // < rows_cap: the grid has ceil(rows_cap / BM) row tiles
  const int n0 = tx * BN;
  const int kb0 = tz * k_per_split;
  const int ke = min(K, kb0 + k_per_split);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int lr = lane & 15, lk = (lane >> 4) * 8;

  // STAGES register sets: the global loads of step k + STAGES*BK are issued
  // right after step k's tiles reach LDS.  One set: two or three lowered the
  // occupancy and gained at most 5-10 % of a launch at 64 rows and fewer, nothing
  // above.  (The loop over sets and its always true first test stay: written
  // out without them the first loads are sunk below the row-count test and the
  // loop is scheduled otherwise, which made gpt2s and small-batch decode steps
  // 0.7-1 % slower.)
  constexpr int STAGES = 1;
  u32x4_t ra[STAGES][A_PER_T], rw[STAGES][W_PER_T];
#define RG_FETCH(S, KK)                                                                                       \
  _Pragma("unroll") for (int i = 0; i < A_PER_T; ++i) {                                                       \
    const int p = tid + i * NT;                                                                               \
    const int plane = p / A_PIECES, q = p % A_PIECES;                                                         \
    const int row = min(m0 + q / (BK / 8), rows_cap - 1); /* rows past M are computed, never stored */       \
    ra[S][i] = *reinterpret_cast<const u32x4_t*>(A + plane * a_plane + (int64_t)row * lda + (KK) + (q % (BK / 8)) * 8); \
  }                                                                                                           \
  _Pragma("unroll") for (int i = 0; i < W_PER_T; ++i) {                                                       \
    const int p = tid + i * NT;                                                                               \
    const int col = min(n0 + p / (BK / 8), N - 1);                                                            \
    rw[S][i] = load_w<NTW>(W + (int64_t)col * ldw + (KK) + (p % (BK / 8)) * 8);                               \
  }
#define RG_STASH(S)                                                                                           \
  _Pragma("unroll") for (int i = 0; i < A_PER_T; ++i) {                                                       \
    const int p = tid + i * NT;                                                                               \
    const int plane = p / A_PIECES, q = p % A_PIECES;                                                         \
    *reinterpret_cast<u32x4_t*>(&sA[plane][(q / (BK / 8)) * LROW + (q % (BK / 8)) * 8]) = ra[S][i];          \
  }                                                                                                           \
  _Pragma("unroll") for (int i = 0; i < W_PER_T; ++i) {                                                       \
    const int p = tid + i * NT;                                                                               \
    *reinterpret_cast<u32x4_t*>(&sW[(p / (BK / 8)) * LROW + (p % (BK / 8)) * 8]) = rw[S][i];                 \
  }

  f32x4_t acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (kb0 + s * BK < ke) { RG_FETCH(s, kb0 + s * BK) }
  // keeps the loads above in front of the row-count test (no sinking past it)
  __asm__ volatile("" ::: "memory");
  const int M = min(rows_now, rows_cap);
  if (m0 >= M) return;
  __shared__ __attribute__((aligned(16))) float s_inv[BM], s_ssq[EPI == GEMM_EPI_RESIDUAL ? BM * WAVES_N : 1];
  RowScale<BM, NT> scale;
  if constexpr (kScaled<EPI>) scale.load(ep, m0, rows_cap, tid);
  for (int k = kb0; k < ke; k += STAGES * BK) {
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
      const int kk = k + s * BK;
      if (kk < ke) {
        __syncthreads();          // the previous step's fragment reads are done
        RG_STASH(s)
        __syncthreads();
        if (kk + STAGES * BK < ke) { RG_FETCH(s, kk + STAGES * BK) }
#pragma unroll
        for (int ks = 0; ks < BK; ks += 32) {
          bf16x8_t bw[WN];
#pragma unroll
          for (int j = 0; j < WN; ++j) bw[j] = lds_frag(&sW[((wn * WN + j) * 16 + lr) * LROW + ks + lk]);
#pragma unroll
          for (int i = 0; i < WM; ++i) {
            const int arow = (wm * WM + i) * 16 + lr;
            const bf16x8_t ah = lds_frag(&sA[0][arow * LROW + ks + lk]);
            const bf16x8_t al = lds_frag(&sA[1][arow * LROW + ks + lk]);
#pragma unroll
            for (int j = 0; j < WN; ++j) {
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bw[j], acc[i][j], 0, 0, 0);
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bw[j], acc[i][j], 0, 0, 0);
            }
          }
        }
      }
    }
  }
#undef RG_FETCH
#undef RG_STASH

  if constexpr (kScaled<EPI>) {
    scale.finish(ep, m0, rows_cap, tid, s_inv);
    scale_rows<WM, WN>(acc, s_inv, wm, lane);
  }
  acc_epilogue<EPI, BM, WM, WN, WAVES_N>(acc, ep, tz, tx, m0, n0, M, N, wm, wn, tid, s_ssq);
}

// 16 bytes per lane from global memory straight into LDS: lane l's piece lands
// at byte address lds + 16 l.  Issued from assembly, so that the compiler does
// not drain every load in flight ahead of each LDS read (it cannot tell the
// buffers apart); the kernel places the waits itself.  No register is written.
__device__ __forceinline__ void dma16(uint32_t lds, uint32_t voff, const bf16_t* sbase) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(sbase)
               : "memory", "m0");
}

// Large tiles: BM x BN output, eight waves, K steps of 64 through two LDS
// buffers that are filled by direct global-to-LDS loads.  A wave keeps the
// fragments of two 32-wide half steps in registers: while it multiplies one
// half it reads the other, and the barrier that hands the buffers over sits
// between the halves of a step, so neither the barrier nor an LDS read waits
// ahead of the MFMAs, and a buffer's loads have a whole step to arrive.  LDS
// rows are 128 bytes, the 16-byte chunk c of row r at c ^ (r / 2 % 8): the 16
// rows of a fragment read cover all 64 banks (the loads permute their global
// chunk within the row's 128 bytes to match).
//
// What bounds it: power.  At 16384 x 17920 x 1536 the MFMAs take 70 % of the
// cycles, at a clock that falls to 1.6-2.0 GHz; 1.11 PFLOP/s issued (two planes)
// against 1.06 for register-staged 256 x 256 tiles, at any schedule, MFMA shape
// or wave tile tried.  The gain is in the smaller tile: the 1536 columns of
// the O and down projections make 768 blocks of 128 x 256 (3 per CU) instead of
// 384 of 256 x 256 (1.5, so 2 rounds): down at 16384 rows 1019 -> 805 us, at
// 4096 rows 441 -> 214; gate/up at 1100 x 768 -> 6144 49.7 -> 25.7.
template <int BM, int BN, int WM, int WN, int EPI>
__global__ __launch_bounds__(512, 2) void k_gemm_dma(const int* __restrict__ d_rows, const bf16_t* __restrict__ A,
                                                     const bf16_t* __restrict__ W, int64_t a_plane, int lda, int ldw,
                                                     int rows_cap, int N, int K, int k_per_split, int gx, int gy,
                                                     GemmEpi ep) {
  constexpr int CH = BK / 8;                                 // 16-byte chunks per row and step
  constexpr int WAVES_N = BN / (16 * WN), NT = 512;
  static_assert((BM / (16 * WM)) * WAVES_N == 8, "eight waves");
  constexpr int A_P = BM * CH / NT, W_P = BN * CH / NT;      // pieces per thread of one A plane, of W
  static_assert((BM * CH) % NT == 0 && (BN * CH) % NT == 0, "tile pieces must split evenly over threads");
  static_assert((EPI != GEMM_EPI_SWIGLU && EPI != GEMM_EPI_QKV) || WN % 2 == 0, "pairs of adjacent column tiles");
  constexpr int STAGE = (2 * BM + BN) * BK;                  // elements: A hi, A lo, W
  __shared__ __attribute__((aligned(128))) bf16_t sm[2 * STAGE];
  const int rows_now = *d_rows;

  // A 1-D grid of a multiple of 8 blocks, dealt to the 8 XCDs in turn: XCD x =
  // b % 8 takes the contiguous tile range [x*per, (x+1)*per) (split-major),
  // walked in groups of TILE_GROUP row tiles.  Within a group the row tiles of one
  // column tile are consecutive, so the blocks that an XCD runs at once share A
  // rows and W columns in its L2.
  constexpr int TILE_GROUP = 4;
  const int per = gridDim.x / 8;
  int w = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (w >= gx * gy * k_split_count(K, k_per_split)) return;
  const int tz = w / (gx * gy);
  w -= tz * gx * gy;
  const int gsz = TILE_GROUP * gx;
  const int g = w / gsz, r0 = g * TILE_GROUP;
  const int rows_g = min(TILE_GROUP, gy - r0);
  const int wi = w - g * gsz;
  const int ty = r0 + wi % rows_g, tx = wi / rows_g;
  const int m0 = ty * BM, n0 = tx * BN;
  const int M = min(rows_now, rows_cap);
  if (m0 >= M) return;
  const int kb0 = tz * k_per_split;
  const int nk = (min(K, kb0 + k_per_split) - kb0) / BK;     // K steps, at least 1

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int lr = lane & 15, lg = lane >> 4;
  // byte offsets of this thread's pieces from the tile's first row (rows past
  // the launch's bound and columns past N read the last one, never stored)
  uint32_t ao[A_P], wo[W_P];
#pragma unroll
  for (int i = 0; i < A_P; ++i) {
    const int p = i * NT + tid, row = p / CH, ch = (p % CH) ^ ((row >> 1) & 7);
    ao[i] = (uint32_t)(min(row, rows_cap - 1 - m0) * lda + ch * 8) * 2;
  }
#pragma unroll
  for (int i = 0; i < W_P; ++i) {
    const int p = i * NT + tid, row = p / CH, ch = (p % CH) ^ ((row >> 1) & 7);
    wo[i] = (uint32_t)(min(row, N - 1 - n0) * ldw + ch * 8) * 2;
  }
  const bf16_t* ah = A + (int64_t)m0 * lda + kb0;            // advance one step per issue
  const bf16_t* al = ah + a_plane;
  const bf16_t* wb = W + (int64_t)n0 * ldw + kb0;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)sm + wave * 1024;
  auto issue = [&](int buf) {
    const uint32_t lb = lds0 + buf * STAGE * 2;
#pragma unroll
    for (int i = 0; i < A_P; ++i) dma16(lb + i * NT * 16, ao[i], ah);
#pragma unroll
    for (int i = 0; i < A_P; ++i) dma16(lb + BM * BK * 2 + i * NT * 16, ao[i], al);
#pragma unroll
    for (int i = 0; i < W_P; ++i) dma16(lb + 2 * BM * BK * 2 + i * NT * 16, wo[i], wb);
    ah += BK;
    al += BK;
    wb += BK;
  };
  const int sl[2] = {lr * BK + (lg ^ ((lr >> 1) & 7)) * 8, lr * BK + ((4 + lg) ^ ((lr >> 1) & 7)) * 8};
  const int abase = wm * WM * 16 * BK, wbase = 2 * BM * BK + wn * WN * 16 * BK;
  bf16x8_t fh[2][WM], fl[2][WM], fw[2][WN];
  f32x4_t acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // half h of buffer buf into fragment set h
#define RG_READ(H, BUF)                                                                                       \
  {                                                                                                           \
    const bf16_t* sb = sm + (BUF) * STAGE + sl[H];                                                            \
    _Pragma("unroll") for (int j = 0; j < WN; ++j) fw[H][j] = lds_frag(sb + wbase + j * 16 * BK);             \
    _Pragma("unroll") for (int i = 0; i < WM; ++i) {                                                          \
      fh[H][i] = lds_frag(sb + abase + i * 16 * BK);                                                          \
      fl[H][i] = lds_frag(sb + abase + BM * BK + i * 16 * BK);                                                \
    }                                                                                                         \
  }
#define RG_MULTIPLY(H)                                                                                        \
  _Pragma("unroll") for (int i = 0; i < WM; ++i) {                                                            \
    _Pragma("unroll") for (int j = 0; j < WN; ++j)                                                            \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fh[H][i], fw[H][j], acc[i][j], 0, 0, 0);         \
    _Pragma("unroll") for (int j = 0; j < WN; ++j)                                                            \
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fl[H][i], fw[H][j], acc[i][j], 0, 0, 0);         \
  }
  // spreads the reads over the MFMAs: one read, two MFMAs, then the rest
#define RG_MIX()                                                                                              \
  _Pragma("unroll") for (int q = 0; q < 2 * WM + WN; ++q) {                                                   \
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                                        \
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);                                                        \
  }                                                                                                           \
  __builtin_amdgcn_sched_group_barrier(0x008, 2 * WM * WN, 0);
  __shared__ __attribute__((aligned(16))) float s_inv[BM], s_ssq[EPI == GEMM_EPI_RESIDUAL ? BM * WAVES_N : 1];
  RowScale<BM, NT> scale;
  if constexpr (kScaled<EPI>) scale.load(ep, m0, rows_cap, tid);   // older than the tiles: covered by their waits
  issue(0);
  if (nk > 1) {
    issue(1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * A_P + W_P) : "memory");   // step 0 has arrived, step 1 may not have
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  RG_READ(0, 0)
  int buf = 0;
  for (int k = 0; k < nk; ++k) {
    __builtin_amdgcn_sched_barrier(0);
    RG_READ(1, buf)
    RG_MULTIPLY(0)
    RG_MIX()
    __builtin_amdgcn_sched_barrier(0);
    // this wave has read all of step k and its share of step k + 1 has arrived
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                 // ... and so has everyone's
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (k + 2 < nk) issue(buf);
    buf ^= 1;
    if (k + 1 < nk) RG_READ(0, buf)
    RG_MULTIPLY(1)
    RG_MIX()
  }
#undef RG_READ
#undef RG_MULTIPLY
#undef RG_MIX
  if constexpr (kScaled<EPI>) {
    scale.finish(ep, m0, rows_cap, tid, s_inv);
    scale_rows<WM, WN>(acc, s_inv, wm, lane);
  }
  acc_epilogue<EPI, BM, WM, WN, WAVES_N>(acc, ep, tz, tx, m0, n0, M, N, wm, wn, tid, s_ssq);
}

// Residual add of the split partials, the next norm's operand x * gain and the
// row's partial sum of squares: one block of 256 threads per (256 columns,
// row), a column per thread.  A thread issues its x and gain loads and a batch
// of its split partials before the first add; blocks of rows past the count (r
// < the launch's row bound, inside every buffer) run the same loads and sums
// but store nothing, so no load waits for the count.  The sums run in split
// order, as in split_sum.
__global__ __launch_bounds__(256) void k_split_residual(const int* __restrict__ d_rows, float* __restrict__ part,
                                                        int64_t pst, float* __restrict__ x,
                                                        const float* __restrict__ norm_g, int N, int S, int ldx,
                                                        GemmEpi ep) {
  __shared__ float red[4];
  const int r = blockIdx.y, c = blockIdx.x * 256 + threadIdx.x, cl = min(c, N - 1);
  const int rows_now = *d_rows;
  const float x0 = x[(int64_t)r * ldx + cl], g = norm_g[cl];
  ep.part = part;          // the preloaded copies
  ep.part_stride = pst;
  const float xv = x0 + split_sum(ep, S, (int64_t)r * N + cl);
  const bool live = r < rows_now && c < N;
  if (live) {
    x[(int64_t)r * ldx + c] = xv;
    act_store<1>(ep.norm_out, (int64_t)r * N + c, xv * g);
  }
  const float ss = wave_sum(c < N ? xv * xv : 0.f);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0 && r < rows_now)
    ep.ssq_out[(int64_t)r * ep.ssq_ld + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// QKV epilogue of split partials for bf16 models, 16 bytes at a time: thread
// u of row r owns packed columns c..c+3 (c = 32 (u / 4) + 4 (u % 4), in the
// lower half of a 32-column group) and their rotation partners c+16..c+19.
// The partials of both column quads are summed in split order (as split_sum),
// rotated, and written as one 16-byte q piece per half or one 8-byte key piece
// per half (values: their transposed layout, one element at a time); one wave per 64 quads of a row.
__global__ __launch_bounds__(64) void k_qkv_epilogue4(const int* __restrict__ d_rows, const float* __restrict__ part,
                                                      int64_t pst, int N, int S, GemmEpi ep) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  constexpr int BATCH = 16;
  const int r = blockIdx.y;
  const int u = blockIdx.x * 64 + threadIdx.x;
  const int rows_now = *d_rows;   // waited for after the partials' loads
  __builtin_assume(S >= 1);
  const int uc = min(u, N / 8 - 1);   // a quad in range: u's own test comes after the loads
  const int c = (uc >> 2) * 32 + (uc & 3) * 4;
  const int hd = ep.hd, half = hd / 2;
  const int head = c / hd, p = c % hd, d = (p >> 5) * 16 + (p & 15);
  const f4* pr = reinterpret_cast<const f4*>(part + (int64_t)r * N + c);
  const int64_t pst4 = pst / 4;
  const float inv = wave_row_scale(ep, r, threadIdx.x);
  f4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < S; s0 += BATCH) {
    f4 ta[BATCH], tb[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      ta[j] = s0 + j < S ? pr[(s0 + j) * pst4] : f4{0.f, 0.f, 0.f, 0.f};
      tb[j] = s0 + j < S ? pr[(s0 + j) * pst4 + 4] : f4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      a += ta[j];
      b += tb[j];
    }
  }
  // a row past the count has no position or page yet
  if (r >= rows_now || u >= N / 8) return;
  a *= inv;
  b *= inv;
  const int pos = ep.row_pos[r];
  bf16_t* pool = (bf16_t*)ep.kv_pool;
  const int n_rot = ep.n_q + ep.n_kv;
  if (head >= n_rot) {                               // value head: no rotation, V^T layout
    const int page = ep.page_tab[(int64_t)ep.row_tab[r] * ep.tab_stride + pos / 16];
    bf16_t* vb = pool + (int64_t)page * ep.geom.page_stride + (int64_t)ep.layer * ep.geom.layer_stride +
                 ((int64_t)ep.n_kv + head - n_rot) * 16 * hd;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      vb[kv_v_off(pos & 15, d + e, hd)] = f32_to_bf16(a[e]);
      vb[kv_v_off(pos & 15, d + e + half, hd)] = f32_to_bf16(b[e]);
    }
    return;
  }
  const f4 co = *reinterpret_cast<const f4*>(ep.rope_cos + (int64_t)pos * half + d);
  const f4 si = *reinterpret_cast<const f4*>(ep.rope_sin + (int64_t)pos * half + d);
  f4 ra, rb;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    ra[e] = a[e] * co[e] - b[e] * si[e];
    rb[e] = b[e] * co[e] + a[e] * si[e];
  }
  if (head < ep.n_q) {
    float* qo = ep.q_out + ((int64_t)r * ep.n_q + head) * hd;
    *reinterpret_cast<f4*>(qo + d) = ra;
    *reinterpret_cast<f4*>(qo + d + half) = rb;
  } else {
    const int page = ep.page_tab[(int64_t)ep.row_tab[r] * ep.tab_stride + pos / 16];
    bf16_t* kp = pool + (int64_t)page * ep.geom.page_stride + (int64_t)ep.layer * ep.geom.layer_stride +
                 (int64_t)(head - ep.n_q) * 16 * hd;
    uint2 ka, kb;
    ka.x = (uint32_t)f32_to_bf16(ra[0]) | ((uint32_t)f32_to_bf16(ra[1]) << 16);
    ka.y = (uint32_t)f32_to_bf16(ra[2]) | ((uint32_t)f32_to_bf16(ra[3]) << 16);
    kb.x = (uint32_t)f32_to_bf16(rb[0]) | ((uint32_t)f32_to_bf16(rb[1]) << 16);
    kb.y = (uint32_t)f32_to_bf16(rb[2]) | ((uint32_t)f32_to_bf16(rb[3]) << 16);
    *reinterpret_cast<uint2*>(kp + kv_k_off(pos & 15, d)) = ka;
    *reinterpret_cast<uint2*>(kp + kv_k_off(pos & 15, d + half)) = kb;
  }
}

// Sum of split partials + SWIGLU or (without a next norm) RESIDUAL epilogue: one
// block of 128 threads (SWIGLU: 64) per (128 columns, row).  Sums the partials
// (all inside the partial buffer; columns past N read a column in range) before
// testing row and column, so the loads wait neither for the row count nor for a
// test of a kernel argument.
template <int EPI>
__global__ __launch_bounds__(128) void k_split_epilogue(const int* __restrict__ d_rows, float* __restrict__ part,
                                                        int64_t pst, int N, int S, GemmEpi ep) {
  const int r = blockIdx.y;
  const int rows_now = *d_rows;
  ep.part = part;          // the preloaded copies
  ep.part_stride = pst;
  if constexpr (EPI == GEMM_EPI_SWIGLU) {
    const int q = threadIdx.x;                                     // 64 threads: a pair of columns each
    const int gc = blockIdx.x * 128 + (q >> 4) * 32 + (q & 15);   // gate column; up is 16 further
    const int gl = min(gc, N - 17);                                // gc itself while in range (N % 32 == 0)
    const float inv = wave_row_scale(ep, r, threadIdx.x);
    const float gt = split_sum(ep, S, (int64_t)r * N + gl) * inv;
    const float up = split_sum(ep, S, (int64_t)r * N + gl + 16) * inv;
    if (r >= rows_now || gc >= N) return;
    act_store<1>(ep.act, (int64_t)r * ep.act_ld + (gc >> 5) * 16 + (q & 15), gt / (1.0f + expf(-gt)) * up);
  } else {
    const int c = blockIdx.x * 128 + threadIdx.x;
    const float v = split_sum(ep, S, (int64_t)r * N + min(c, N - 1));
    if (r >= rows_now || c >= N) return;
    ep.x[(int64_t)r * ep.ldx + c] += v;
  }
}

// fp32 models: v_mfma_f32_16x16x4_f32 (full fp32 products and sums).  A block
// owns 16 WMT rows x 32 columns; its four waves split K in turns of 16 and
// meet in LDS, where the partial sums are added in wave order and the
// epilogue runs.  Lane (l % 16, l / 16) loads four consecutive k's of its row
// and column (16 bytes, 64 contiguous bytes per row); MFMA j of a turn takes
// the j-th of each, the same k on both sides.  These launches are small (fp32
// is the toy decoder's type): what counts is the length of the load chain.  A
// thread per output walking K alone took 22.9 us a launch in the 128-wide
// decoder's decode step and needed a second launch for the epilogue; this
// takes 3.6-4.6 us with it.
template <int WMT, int EPI>
__global__ __launch_bounds__(256) void k_gemm_f32(const float* __restrict__ A, const float* __restrict__ W,
                                                  const int* __restrict__ d_rows, int lda, int ldw, int rows_cap,
                                                  int N, int K, GemmEpi ep) {
  constexpr int BM = 16 * WMT;
  __shared__ float red[4][BM][33];
  __shared__ float s_inv[BM];
  const int rows_now = *d_rows;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lk = (lane >> 4) * 4;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * 32;
  RowScale<BM, 256> scale;
  if constexpr (kScaled<EPI>) scale.load(ep, m0, rows_cap, tid);
  const float* wp[2];
  const float* ap[WMT];
#pragma unroll
  for (int j = 0; j < 2; ++j) wp[j] = W + (int64_t)min(n0 + j * 16 + lr, N - 1) * ldw + lk;
#pragma unroll
  for (int i = 0; i < WMT; ++i) ap[i] = A + (int64_t)min(m0 + i * 16 + lr, rows_cap - 1) * lda + lk;
  f32x4_t acc[WMT][2];
#pragma unroll
  for (int i = 0; i < WMT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // U turns' loads are issued before the first product; turns past K read the
  // last one again and are skipped
  constexpr int U = WMT == 1 ? 4 : 2;
  for (int k = wave * 16; k < K; k += 64 * U) {
    f32x4_t w[U][2], a[U][WMT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = min(k + 64 * u, K - 16);
#pragma unroll
      for (int j = 0; j < 2; ++j) w[u][j] = *reinterpret_cast<const f32x4_t*>(wp[j] + kk);
#pragma unroll
      for (int i = 0; i < WMT; ++i) a[u][i] = *reinterpret_cast<const f32x4_t*>(ap[i] + kk);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + 64 * u < K) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < WMT; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][e], w[u][j][e], acc[i][j], 0, 0, 0);
      }
  }
#pragma unroll
  for (int i = 0; i < WMT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][i * 16 + (lane >> 4) * 4 + e][j * 16 + lr] = acc[i][j][e];
  __syncthreads();
  const int M = min(rows_now, rows_cap);
  if constexpr (kScaled<EPI>) scale.finish(ep, m0, rows_cap, tid, s_inv);
  for (int i = tid; i < BM * 16; i += 256) {   // columns c and c + 16 of a row: 16 neighbouring lanes a row
    const int rr = i >> 4, cc = i & 15, r = m0 + rr, c = n0 + cc;
    const bool on0 = r < M && c < N, on1 = r < M && c + 16 < N;
    const float inv = kScaled<EPI> ? s_inv[rr] : 1.f;
    const float v0 = inv * ((red[0][rr][cc] + red[1][rr][cc]) + (red[2][rr][cc] + red[3][rr][cc]));
    const float v1 = inv * ((red[0][rr][cc + 16] + red[1][rr][cc + 16]) + (red[2][rr][cc + 16] + red[3][rr][cc + 16]));
    if constexpr (EPI == GEMM_EPI_QKV) {
      if (on0) qkv_store_f32(ep, r, c, v0, v1);
    } else if constexpr (EPI == GEMM_EPI_SWIGLU) {
      if (on0) act_store<0>(ep.act, (int64_t)r * ep.act_ld + (n0 >> 1) + cc, v0 / (1.0f + expf(-v0)) * v1);
    } else if constexpr (EPI == GEMM_EPI_RESIDUAL) {
      float* xp = ep.x + (int64_t)r * ep.ldx + c;
      const float x0 = on0 ? xp[0] + v0 : 0.f, x1 = on1 ? xp[16] + v1 : 0.f;
      if (on0) xp[0] = x0;
      if (on1) xp[16] = x1;
      if (ep.norm_g) {
        if (on0) act_store<0>(ep.norm_out, (int64_t)r * N + c, x0 * ep.norm_g[c]);
        if (on1) act_store<0>(ep.norm_out, (int64_t)r * N + c + 16, x1 * ep.norm_g[c + 16]);
        float ss = fmaf(x0, x0, x1 * x1);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
        if (cc == 0 && r < M) ep.ssq_out[(int64_t)r * ep.ssq_ld + blockIdx.x] = ss;
      }
    } else {
      if (on0) ep.C[(int64_t)r * ep.ldc + c] = v0;
      if (on1) ep.C[(int64_t)r * ep.ldc + c + 16] = v1;
    }
  }
}

template <int WMT>
hipError_t launch_f32(const float* A, int lda, const float* W, int ldw, const int* d_rows, int rows_ub, int N, int K,
                      const GemmEpi& ep, hipStream_t st) {
  const dim3 grid((N + 31) / 32, (rows_ub + 16 * WMT - 1) / (16 * WMT));
#define RG_F32(E) hipLaunchKernelGGL((k_gemm_f32<WMT, E>), grid, dim3(256), 0, st, A, W, d_rows, lda, ldw, rows_ub, N, K, ep)
  switch (ep.mode) {
    case GEMM_EPI_STORE: RG_F32(GEMM_EPI_STORE); break;
    case GEMM_EPI_RESIDUAL: RG_F32(GEMM_EPI_RESIDUAL); break;
    case GEMM_EPI_SWIGLU: RG_F32(GEMM_EPI_SWIGLU); break;
    case GEMM_EPI_QKV: RG_F32(GEMM_EPI_QKV); break;
    default: return hipErrorInvalidValue;
  }
#undef RG_F32
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN>
hipError_t launch_tiled(const void* A, int lda, int64_t a_plane, const void* W, int ldw, const int* d_rows,
                        int rows_ub, int N, int K, int splits, int k_per_split, const GemmEpi& ep, hipStream_t st) {
  constexpr int NT = (BM / (16 * WM)) * (BN / (16 * WN)) * 64;
  const int gx = (N + BN - 1) / BN, gy = (rows_ub + BM - 1) / BM;
  const dim3 grid(gx, gy, splits);
  // One row tile: every weight piece is read by one block only, so its loads
  // are non-temporal.  With several row tiles the weight tiles are re-read
  // by the other row tiles' blocks through L2, and non-temporal loads there
  // measured 12 % slower over the 1.5B group step.
  const bool ntw = gy == 1;
#define RG_TILED_K(E, NTV)                                                                                    \
  hipLaunchKernelGGL((k_gemm_tiled<BM, BN, WM, WN, E, NTV>), grid, dim3(NT), 0, st, (const bf16_t*)A,          \
                     (const bf16_t*)W, d_rows, a_plane, lda, ldw, rows_ub, N, K, k_per_split, ep)
#define RG_TILED(E)                                                                                           \
  do {                                                                                                        \
    if (ntw) RG_TILED_K(E, true);                                                                             \
    else RG_TILED_K(E, false);                                                                                \
  } while (0)
  if (splits > 1) {
    RG_TILED(GEMM_EPI_PARTIAL);
  } else {
    switch (ep.mode) {
      case GEMM_EPI_STORE: RG_TILED(GEMM_EPI_STORE); break;
      case GEMM_EPI_RESIDUAL: RG_TILED(GEMM_EPI_RESIDUAL); break;
      case GEMM_EPI_SWIGLU: RG_TILED(GEMM_EPI_SWIGLU); break;
      case GEMM_EPI_QKV: RG_TILED(GEMM_EPI_QKV); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef RG_TILED
#undef RG_TILED_K
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN>
hipError_t launch_dma(const void* A, int lda, int64_t a_plane, const void* W, int ldw, const int* d_rows, int rows_ub,
                      int N, int K, int splits, int k_per_split, const GemmEpi& ep, hipStream_t st) {
  const int gx = (N + BN - 1) / BN, gy = (rows_ub + BM - 1) / BM;
  // byte offsets inside a tile are 32-bit
  if ((int64_t)BM * lda * 2 > UINT32_MAX || (int64_t)BN * ldw * 2 > UINT32_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(((int64_t)gx * gy * splits + 7) / 8 * 8));
#define RG_DMA(E)                                                                                             \
  hipLaunchKernelGGL((k_gemm_dma<BM, BN, WM, WN, E>), grid, dim3(512), 0, st, d_rows, (const bf16_t*)A,       \
                     (const bf16_t*)W, a_plane, lda, ldw, rows_ub, N, K, k_per_split, gx, gy, ep)
  if (splits > 1) {
    RG_DMA(GEMM_EPI_PARTIAL);
  } else {
    switch (ep.mode) {
      case GEMM_EPI_STORE: RG_DMA(GEMM_EPI_STORE); break;
      case GEMM_EPI_RESIDUAL: RG_DMA(GEMM_EPI_RESIDUAL); break;
      case GEMM_EPI_SWIGLU: RG_DMA(GEMM_EPI_SWIGLU); break;
      case GEMM_EPI_QKV: RG_DMA(GEMM_EPI_QKV); break;
      case GEMM_EPI_LOGPROB:
        if (ep.lse_ld < gx * (BN / (16 * WN))) return hipErrorInvalidValue;
        RG_DMA(GEMM_EPI_LOGPROB);
        break;
      default: return hipErrorInvalidValue;
    }
  }
#undef RG_DMA
  return hipGetLastError();
}

hipError_t launch_split_epilogue(const int* d_rows, int rows_ub, int N, int S, const GemmEpi& ep, hipStream_t st) {
  if (ep.mode == GEMM_EPI_RESIDUAL && ep.norm_g) {
    hipLaunchKernelGGL(k_split_residual, dim3((N + 255) / 256, rows_ub), dim3(256), 0, st, d_rows, ep.part,
                       ep.part_stride, ep.x, ep.norm_g, N, S, ep.ldx, ep);
    return hipGetLastError();
  }
  dim3 grid((N + 127) / 128, rows_ub);
  switch (ep.mode) {
    case GEMM_EPI_RESIDUAL:
      hipLaunchKernelGGL((k_split_epilogue<GEMM_EPI_RESIDUAL>), grid, dim3(128), 0, st, d_rows, ep.part,
                         ep.part_stride, N, S, ep);
      break;
    case GEMM_EPI_SWIGLU:
      hipLaunchKernelGGL((k_split_epilogue<GEMM_EPI_SWIGLU>), grid, dim3(64), 0, st, d_rows, ep.part, ep.part_stride,
                         N, S, ep);
      break;
    case GEMM_EPI_QKV:
      hipLaunchKernelGGL(k_qkv_epilogue4, dim3((N / 8 + 63) / 64, rows_ub), dim3(64), 0, st, d_rows, ep.part,
                         ep.part_stride, N, S, ep);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The register-staged tiles, for row counts where a launch streams weights
// rather than fills the MFMAs.  Tile rows, measured over the projection shapes
// at 32..512 rows: the smallest tiles win while they keep the block count
// moderate (more, shorter blocks balance the CUs better); wide outputs with
// many rows take 64-row tiles, and the widest at 65-128 rows none of these
// (0: the direct-to-LDS tiles).  The tile shape does not change any result:
// every output still accumulates K in the same order.
int staged_tile_rows(int rows_ub, int N) {
  if (rows_ub <= 16) return 16;
  const int64_t ct = (N + 127) / 128;
  const int64_t c32 = ct * ((rows_ub + 31) / 32), c64 = ct * ((rows_ub + 63) / 64);
  if (c64 > 2048) return rows_ub <= 64 ? 64 : 0;
  if (c32 > 2048 || (rows_ub > 128 && c32 > 600)) return 64;
  return 32;
}

constexpr int64_t kNoSplitBlocks = 256;   // staged tiles split K below this many output tiles

// 32-row tiles take 64 columns where that measured faster in the rollout (1.5B
// and 7B group steps, ms per row bucket):
// * wide outputs (gate/up) at 33-64 rows when 128-column tiles leave fewer
//   than two blocks per CU (1.5B: 280 blocks -> 560, 644 -> 571 ms; 7B's
//   592 blocks measured slower at 1,184);
// * narrow outputs at 17-64 rows, and at 65-128 rows those with K <= 2N (QKV,
//   O), while the 64-column tiles still number fewer than the no-split
//   threshold: the same block count then needs half the split-K factor and the
//   split reduction reads half the partials (1.5B at 64 rows: QKV + O + down
//   1096 -> 993 ms; at 128 rows QKV + O 702 -> 643 ms).  7B's QKV at 128 rows
//   would cross the threshold and run unsplit, 1.6x slower;
// * the unsplit QKV (N > K) at 512 rows and more (1.5B: 512 -> 471 ms).
// All others 128 columns.  A tile shape that changes the split factor
// changes where the fp32 split sums are cut, so results move within fp32
// rounding.
int staged_tile_cols(int bm, int rows_ub, int N, int K) {
  if (bm == 32) {
    const int64_t row_tiles = (rows_ub + 31) / 32;
    if (N >= 8192)
      return rows_ub > 32 && rows_ub <= 64 && (int64_t)((N + 127) / 128) * row_tiles < 2 * kNoSplitBlocks ? 64 : 128;
    const bool splits64 = (int64_t)((N + 63) / 64) * row_tiles < kNoSplitBlocks;
    if (rows_ub <= 64 && splits64) return 64;
    if (rows_ub <= 128 && K <= 2 * N && splits64) return 64;
    if (rows_ub >= 512 && N > K) return 64;
  }
  return 128;
}

// Widths of the direct-to-LDS tiles and the time of one 64-wide K step of a
// 128-row tile with every CU busy (us, measured at 16384 x 37888 x 3584).
constexpr int kDmaCols[4] = {128, 192, 256, 320};
constexpr double kDmaStep[4] = {1.09, 1.40, 1.61, 1.97};

// Tile width and split of a direct-to-LDS launch: the cheapest by rounds of
// 256 blocks x (steps x step time + 4 us), plus, when K is split, 4 us and the
// partials' write and read at 8 TB/s for the reduction.  Against measured
// times (us, model / measured): 512 x 1536 x 8960 256 columns split 10 38 /
// 38, 192 split 8 40 / 40, 128 split 5 42 / 45; 256 x 3584 x 18944 256 split 9
// 70 / 74, 192 split 6 84 / 88, 128 split 4 96 / 99; and it ranks the widths
// as measured at every shape tried unsplit (512 x 17920 x 1536: 320 columns
// 56 us, 256 79; 256 rows: 192 39, 256 43; 8191 x 1536 x 8960: 192 416, 256
// 432; 4096 x 768 x 3072: 128 47, 256 69).
GemmPlan dma_plan(int rows_ub, int N, int K, int max_splits) {
  GemmPlan best{128, 0, true, 1, K};
  double best_t = 0.0;
  const int64_t gy = ceil_div(rows_ub, 128);
  for (int c = 0; c < 4; ++c) {
    const int64_t tiles = gy * ceil_div(N, kDmaCols[c]);
    for (int want = 1; want <= std::max(1, std::min(max_splits, K / 256)); ++want) {
      const int kps = (int)(ceil_div(ceil_div(K, want), 64) * 64), S = (int)ceil_div(K, kps);
      double t = (double)ceil_div(tiles * S, 256) * (kps / 64 * kDmaStep[c] + 4.0);
      if (S > 1) t += 4.0 + (double)S * rows_ub * N / 1e6;
      if (best.bn == 0 || t < best_t) {
        best_t = t;
        best.bn = kDmaCols[c];
        best.splits = S;
        best.k_per_split = kps;
      }
    }
  }
  return best;
}

}  // namespace

// Which tiles.  Direct-to-LDS tiles (128 rows) above 1024 rows, and below that
// where a launch has the MFMA work to fill the chip: 10 GFLOP issued above 128
// rows, 30 at 65-128 (us, direct / staged, reductions included: 512 x 1536 x
// 8960 38 / 57; 256 rows 27 / 31; 256 x 4608 x 3584 31 / 55; 128 x 3584 x
// 18944 49 / 81; but 512 x 1536 x 1536 20 / 19 and 128 x 17920 x 1536 35 / 32).
// Staged tiles split K only while their output tiles leave the chip short of
// blocks, to about 384 blocks (768 for narrow outputs, whose partials are
// small), and only as far as the fp32 partials (written once, read once: 8
// bytes per output element and split) stay within twice the weight bytes or
// 24 MiB.
GemmPlan gemm_plan(int dtype, int rows_ub, int N, int K, int max_splits) {
  if (dtype != 1) return GemmPlan{16, 32, false, 1, K};
  // the split reductions take a row per block in grid dimension y (at most 65535)
  max_splits = rows_ub > 65535 ? 1 : std::max(1, std::min(max_splits, GEMM_MAX_SPLITS));
  const int bm = staged_tile_rows(rows_ub, N);
  const double work = 4.0 * rows_ub * N * K;   // both planes
  if (rows_ub > 1024 || bm == 0 || work >= (rows_ub > 128 ? 10e9 : rows_ub > 64 ? 30e9 : 1e300))
    return dma_plan(rows_ub, N, K, max_splits);
  const int bn = staged_tile_cols(bm, rows_ub, N, K);
  const int64_t blocks = ceil_div(N, bn) * ceil_div(rows_ub, bm);
  int64_t S = 1;
  if (blocks < kNoSplitBlocks) S = ceil_div(N >= 8192 ? 384 : 768, blocks);
  const int64_t budget = std::max<int64_t>(4LL * N * K, 24LL << 20);
  S = std::max<int64_t>(1, std::min<int64_t>({S, K / 128, budget / (8LL * rows_ub * N), max_splits}));
  GemmPlan p{bm, bn, false, 1, K};
  p.k_per_split = (int)(ceil_div(ceil_div(K, S), 64) * 64);
  p.splits = (int)ceil_div(K, p.k_per_split);
  return p;
}

int gemm_ssq_parts(int dtype, const GemmPlan& p, int N) {
  return (int)ceil_div(N, dtype != 1 ? 32 : p.splits > 1 ? 256 : p.bn);
}

int gemm_lse_parts(const GemmPlan& p, int N) { return (int)ceil_div(N, p.bn) * (p.bn == 256 ? 4 : 2); }

hipError_t launch_gemm(int dtype, const GemmPlan& p, const void* A, int lda, int64_t a_plane, const void* W, int ldw,
                       const int* d_rows, int rows_ub, int N, int K, const GemmEpi& ep, hipStream_t st) {
  if (rows_ub <= 0) return hipSuccess;
  const int S = p.splits, kps = p.k_per_split;
  if (S < 1 || S > GEMM_MAX_SPLITS || (S > 1 && !ep.part)) return hipErrorInvalidValue;
  if (S > 1 && (ep.mode == GEMM_EPI_STORE || ep.mode == GEMM_EPI_LOGPROB)) return hipErrorInvalidValue;   // lm head: unsplit
  if ((ep.mode == GEMM_EPI_SWIGLU || ep.mode == GEMM_EPI_QKV) && N % 32) return hipErrorInvalidValue;
  if (ep.mode == GEMM_EPI_QKV && (ep.hd % 32 || 128 % ep.hd)) return hipErrorInvalidValue;
  if (dtype == 1) {
    if (K % BK || kps % BK || N % 16 || k_split_count(K, kps) != S) return hipErrorInvalidValue;
    hipError_t e = hipErrorInvalidValue;
#define RG_TILE(F, ...) e = F<__VA_ARGS__>(A, lda, a_plane, W, ldw, d_rows, rows_ub, N, K, S, kps, ep, st)
    if (p.dma) {
      if (p.bn == 128) RG_TILE(launch_dma, 128, 128, 2, 4);
      else if (p.bn == 192) RG_TILE(launch_dma, 128, 192, 2, 6);
      else if (p.bn == 256) RG_TILE(launch_dma, 128, 256, 4, 4);
      else if (p.bn == 320) RG_TILE(launch_dma, 128, 320, 2, 10);
    } else if (p.bm == 16 && p.bn == 128) {
      RG_TILE(launch_tiled, 16, 128, 1, 2);
    } else if (p.bm == 32 && p.bn == 64) {
      RG_TILE(launch_tiled, 32, 64, 1, 2);
    } else if (p.bm == 32 && p.bn == 128) {
      RG_TILE(launch_tiled, 32, 128, 1, 4);
    } else if (p.bm == 64 && p.bn == 128) {
      RG_TILE(launch_tiled, 64, 128, 2, 4);
    }
#undef RG_TILE
    if (e != hipSuccess || S == 1) return e;
    return launch_split_epilogue(d_rows, rows_ub, N, S, ep, st);
  }
  // fp32: 64-row tiles once 16-row ones give every CU two blocks
  if (S != 1 || K % 16) return hipErrorInvalidValue;
  if ((int64_t)((N + 31) / 32) * ((rows_ub + 15) / 16) > 512)
    return launch_f32<4>((const float*)A, lda, (const float*)W, ldw, d_rows, rows_ub, N, K, ep, st);
  return launch_f32<1>((const float*)A, lda, (const float*)W, ldw, d_rows, rows_ub, N, K, ep, st);
}
