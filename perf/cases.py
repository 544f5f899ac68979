"""The calls that a user of this library makes, as cases to be timed and checked.

A case is a dict of plain values; ``prepare`` makes what a training program
holds before the call (a loaded policy, prompts, finished completions,
rewards), ``run`` is one call through the public entry points, ``work`` what
that call cannot do without, and ``exact`` the same values in 64 bits in plain
torch.

Decoder shapes are those of the repository's workloads (tiny, gpt2s, 1.5b, 7b)
at their full widths.  The deep ones run at a few layers, since every layer
runs the same kernels, and the 7b one with the 32000-token vocabulary of
gpt2s, so that a policy is made in about a second.

Rollouts are teacher-forced (``force_tokens``): the same kernels run as in a
free rollout, but a rounding difference cannot change which token is fed next,
so the log-probabilities of every step can be compared.  Sequence lengths and
group sizes follow from the case alone, so that the work of a case does not
depend on the seed; token ids, weights, rewards and log-probabilities come
from the seed.
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2606_02218_amd as rg

_MODELS = {
    "tiny": dict(d_model=128, n_q_heads=4, n_kv_heads=4, head_dim=32, ffn_dim=512, rope_theta=1e4, dtype="f32"),
    "gpt2s": dict(d_model=768, n_q_heads=12, n_kv_heads=12, head_dim=64, ffn_dim=3072, rope_theta=1e4, dtype="bf16"),
    "1.5b": dict(d_model=1536, n_q_heads=12, n_kv_heads=2, head_dim=128, ffn_dim=8960, rope_theta=1e6, dtype="bf16"),
    "7b": dict(d_model=3584, n_q_heads=28, n_kv_heads=4, head_dim=128, ffn_dim=18944, rope_theta=1e6, dtype="bf16"),
}
_DEFAULTS = {"tiny": (2, 512), "gpt2s": (12, 32000), "1.5b": (4, 151936), "7b": (2, 32000)}   # layers, vocabulary


def _model_case(kind, model, P, plen, G, new, dump=0, temperature=1.0, name=None):
    """plen, G: (lo, hi) ranges, drawn per prompt; new: (median length, spread
    of its logarithm, max_new); dump: steps whose raw logits are returned."""
    layers, vocab = _DEFAULTS[model]
    c = {"name": name} if name else {}
    c.update(kind=kind, model=model, layers=layers, vocab=vocab, prompts=P, plen_lo=plen[0], plen_hi=plen[1],
             g_lo=G[0], g_hi=G[1], len_median=new[0], len_spread=new[1], max_new=new[2], dump=dump,
             temperature=temperature)
    return c


def _score_case(P, G, new, mode, name=None):
    c = {"name": name} if name else {}
    c.update(kind="scores", prompts=P, g_lo=G[0], g_hi=G[1], len_median=new[0], len_spread=new[1], max_new=new[2],
             mode=mode)
    return c


def listed():
    return [
        # The smallest rollout: the fp32 toy decoder of the smoke test and of unit tests in a user's program;
        # 32 steps of tiny kernels, all launches and latency.
        _model_case("rollout", "tiny", 1, (16, 16), (4, 4), (20, 0.4, 32), dump=4, name="rollout_tiny_f32"),
        # A whole small model: 8 prompts x 8, head_dim 64 without GQA, ragged lengths.
        _model_case("rollout", "gpt2s", 8, (256, 256), (8, 8), (80, 0.6, 160), dump=4, name="rollout_gpt2s"),
        # The straggler tail: few sequences left, each step streams the weights for a handful of rows and reads
        # contexts that grow to 2560 positions.
        _model_case("rollout", "1.5b", 2, (512, 512), (4, 4), (1400, 0.4, 2048), dump=8, name="rollout_1.5b_tail"),
        # An effective batch of about a hundred: group sizes as the controller mixes them, odd prompt lengths,
        # a sampling temperature.
        _model_case("rollout", "1.5b", 8, (131, 509), (4, 32), (100, 0.6, 200), dump=2, temperature=0.7,
                    name="rollout_1.5b_dyn"),
        # The full training batch: 32 prompts x 16, the first steps, where every row is alive.
        _model_case("rollout", "1.5b", 32, (512, 512), (16, 16), (60, 0.3, 64), dump=1, name="rollout_1.5b_full"),
        # The larger decoder's widths (7 query heads per kv head), 16 prompts x 16, long prompts.
        _model_case("rollout", "7b", 16, (1024, 1024), (16, 16), (44, 0.3, 48), dump=2, name="rollout_7b"),
        # The prefill of the full batch: 16384 prompt tokens, one sampled token each.
        _model_case("rollout", "1.5b", 32, (512, 512), (16, 16), (1, 0.0, 1), dump=1, name="prefill_1.5b"),
        # One long ragged prompt (the longest context of the workloads is 9216): attention over it, then a few
        # decode steps that read it back.
        _model_case("rollout", "1.5b", 1, (8191, 8191), (16, 16), (8, 0.0, 8), dump=8, name="long_prompt_1.5b"),
        # The loss forward of a step: log-probabilities of finished completions under the current weights.
        _model_case("recompute", "1.5b", 8, (512, 512), (8, 8), (300, 0.6, 1024), name="recompute_1.5b"),
        # The same for the small model, ragged prompts and odd lengths.
        _model_case("recompute", "gpt2s", 8, (37, 256), (3, 8), (150, 0.8, 701), name="recompute_gpt2s"),
        # Everything between the rollout and the update, on a small batch and on the full one: advantage,
        # filter, straggler statistics and the clipped surrogate (sequence mean / token mean).
        _score_case(8, (8, 8), (300, 0.6, 1024), "seq", name="scores_8x8"),
        _score_case(32, (16, 16), (1200, 0.8, 4096), "token", name="scores_32x16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes log-uniform, odd ones among them."""
    pick = rng.choice(["tiny", "gpt2s", "1.5b", "1.5b", "7b", "prefill", "long", "recompute", "recompute", "scores",
                       "scores"])
    temp = rng.choice([1.0, 1.0, 0.7, 1.3])
    if pick == "scores":
        P, g, max_new = _log_int(rng, 8, 64), rng.choice([2, 3, 4, 8, 16]), _log_int(rng, 32, 4096)
        return _score_case(P, (g, rng.randint(g, 16)), (max(1, max_new // 3), rng.uniform(0.3, 0.9), max_new),
                           rng.choice(["token", "seq"]))
    if pick == "recompute":
        model = rng.choice(["tiny", "gpt2s", "1.5b"])
        P, g, max_new = _log_int(rng, 1, 8), rng.randint(1, 4), _log_int(rng, 8, 700)
        lo = _log_int(rng, 8, 400)
        return _model_case("recompute", model, P, (lo, lo + rng.randint(0, 100)), (g, rng.randint(g, 8)),
                           (max(1, max_new // 2), rng.uniform(0.2, 0.8), max_new), temperature=temp)
    if pick == "prefill":
        lo = _log_int(rng, 16, 500)
        return _model_case("rollout", rng.choice(["gpt2s", "1.5b"]), _log_int(rng, 1, 31), (lo, lo + rng.randint(0, 12)),
                           (1, rng.randint(1, 16)), (1, 0.0, 1), dump=1, temperature=temp)
    if pick == "long":
        n = _log_int(rng, 1500, 8000)
        return _model_case("rollout", rng.choice(["gpt2s", "1.5b"]), 1, (n, n), (1, rng.randint(1, 4)), (8, 0.0, 8),
                           dump=8, temperature=temp)
    if pick == "7b":
        lo = _log_int(rng, 64, 1000)
        return _model_case("rollout", "7b", _log_int(rng, 1, 15), (lo, lo + rng.randint(0, 24)),
                           (2, rng.randint(2, 16)), (24, 0.4, 44), dump=2, temperature=temp)
    P = _log_int(rng, 1, 4 if pick == "tiny" else 30)
    most = 16 if pick != "tiny" else 6
    g = rng.randint(1, most)
    max_new = _log_int(rng, 8, max(12, min(160, 2000 // (P * 2))))
    lo = rng.randint(4, 40) if pick == "tiny" else _log_int(rng, 16, 500)
    return _model_case("rollout", pick, P, (lo, lo + rng.randint(0, 12)), (g, rng.randint(g, most)),
                       (max(1, max_new // 2), rng.uniform(0.2, 0.8), max_new), dump=1, temperature=temp)


def _sizes(case):
    """(prompt lengths, group sizes, completion lengths) of a case."""
    r = random.Random(repr(sorted((k, v) for k, v in case.items() if k != "name")))
    P, hi = case["prompts"], case["max_new"]
    lens = [r.randint(case["plen_lo"], case["plen_hi"]) for _ in range(P)] if "plen_lo" in case else None
    if case["g_hi"] >= 4 * case["g_lo"] and case["g_lo"] >= 4:   # the admissible sizes of the dynamic workload
        G = [r.choice([g for g in (4, 8, 16, 32) if case["g_lo"] <= g <= case["g_hi"]]) for _ in range(P)]
    else:
        G = [r.randint(case["g_lo"], case["g_hi"]) for _ in range(P)]
    lo = max(1, case.get("dump", 1))                # every sequence lives through the dumped steps
    L = [min(hi, max(lo, int(case["len_median"] * math.exp(case["len_spread"] * r.gauss(0, 1)) + 0.5)))
         for _ in range(sum(G))]
    return lens, G, L


def _shape(case):
    return SimpleNamespace(n_layers=case["layers"], vocab=case["vocab"], eos_id=case["vocab"] - 1, rms_eps=1e-6,
                           **_MODELS[case["model"]])


def _weights(shape, seed):
    """Matrices ~ N(0, 0.02) on the GPU, rounded to the storage type; norm gains 1 (as the repository's workloads)."""
    gen = torch.Generator(device="cuda").manual_seed(seed * 7919 + 1)
    dt = torch.bfloat16 if shape.dtype == "bf16" else torch.float32

    def mat(n, k):
        return torch.randn(n, k, generator=gen, device="cuda", dtype=torch.float32).mul_(0.02).to(dt)

    d, f, q, kv = shape.d_model, shape.ffn_dim, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim
    layers = [{"wq": mat(q, d), "wk": mat(kv, d), "wv": mat(kv, d), "wo": mat(d, q), "w_gate": mat(f, d),
               "w_up": mat(f, d), "w_down": mat(d, f)} for _ in range(shape.n_layers)]
    return SimpleNamespace(embed=mat(shape.vocab, d), lm_head=mat(shape.vocab, d), layers=layers)


def _host_weights(shape, seed):
    w = _weights(shape, seed)
    ones = np.ones(shape.d_model, np.float32)

    def host(t):
        return t.cpu().float().numpy()

    return SimpleNamespace(embed=host(w.embed), final_norm=ones, lm_head=host(w.lm_head),
                           layers=[dict({k: host(t) for k, t in lw.items()}, attn_norm=ones, ffn_norm=ones)
                                   for lw in w.layers])


def _token_inputs(case, seed):
    """Prompts (a list of device int32 tensors), completions [N, max_new] and their lengths."""
    plen, G, L = _sizes(case)
    rng = np.random.default_rng([seed, 5])
    V, N, T = case["vocab"], sum(G), case["max_new"]
    prompts = [torch.from_numpy(rng.integers(0, V - 1, size=n).astype(np.int32)).cuda() for n in plen]
    tok = rng.integers(0, V - 1, size=(N, T)).astype(np.int32)
    tok[np.arange(N), np.asarray(L) - 1] = V - 1                      # EOS ends a completion
    return prompts, G, np.asarray(L, np.int32), torch.from_numpy(tok).cuda()


def prepare(case, seed):
    if case["kind"] == "scores":
        return _prepare_scores(case, seed)
    shape = _shape(case)
    prompts, G, L, tok = _token_inputs(case, seed)
    plen = [int(p.numel()) for p in prompts]
    pol = rg.Policy(shape, _host_weights(shape, seed), max_seqs=sum(G), max_prompts=len(G),
                    max_prompt_tokens=sum(plen), max_context=max(plen) + case["max_new"])
    return {"case": case, "pol": pol, "prompts": prompts, "G": G, "forced": L, "tok": tok,
            "len": torch.from_numpy(L).cuda(), "seed": seed + 1234}


def _prepare_scores(case, seed):
    _, G, L = _sizes(case)
    rng = np.random.default_rng([seed, 6])
    N, T = sum(G), case["max_new"]
    p = np.repeat(rng.uniform(0.0, 1.0, len(G)).round(1), G)          # some groups all right or all wrong
    valid = np.arange(T)[None, :] < np.asarray(L)[:, None]
    new = np.where(valid, rng.normal(-11.9, 1.0, (N, T)), 0.0).astype(np.float32)
    old = np.where(valid, new + rng.normal(0.0, 0.15, (N, T)), 0.0).astype(np.float32)
    return {"case": case, "rewards": torch.from_numpy((rng.random(N) < p).astype(np.float32)).cuda(),
            "G": torch.tensor(G, dtype=torch.int32, device="cuda"),
            "len": torch.tensor(L, dtype=torch.int32, device="cuda"), "new": torch.from_numpy(new).cuda(),
            "old": torch.from_numpy(old).cuda(), "ctl": rg.Sagc(seed=seed)}


def run(state):
    c = state["case"]
    if c["kind"] == "scores":
        adv = rg.group_advantage(state["rewards"], state["G"])
        keep, kept, n = rg.group_filter(state["rewards"], state["G"])
        stats = state["ctl"].group_stats(state["len"], state["G"])
        loss = rg.grpo_surrogate(state["new"], state["old"], adv, state["len"], state["G"], eps_lo=0.2, eps_hi=0.28,
                                 mode=c["mode"], keep=keep)
        return {"adv": adv, "keep": keep, "kept": kept, "n": n, "stats": stats, "loss": loss}
    if c["kind"] == "recompute":
        return {"lp": state["pol"].recompute_logprobs(state["prompts"], state["G"], state["tok"], state["len"],
                                                      temperature=c["temperature"])}
    tokens, lengths, lp, logits = state["pol"].rollout(
        state["prompts"], state["G"], c["max_new"], state["seed"], temperature=c["temperature"],
        forced_len=state["forced"], force_tokens=state["tok"], dump_steps=c["dump"])
    return {"tokens": tokens, "lengths": lengths, "lp": lp, "logits": logits}


def tolerance(case):
    # Measured against exact(): scores 4e-8 (fp32 results of fp64 sums), tiny 5e-7 (fp32 sums), bf16 models 3.5e-4
    # (logits; a key or value that rounds the other way into the bf16 cache).  Tokens differ at ties only.
    if case["kind"] == "scores":
        return {"rel": 2e-7, "max": 1e-6}
    if case["model"] == "tiny":
        return {"rel": 2e-6, "max": 1e-4, "differ": 1e-2}
    return {"rel": 1.5e-3, "max": 2e-2, "differ": 1e-2}


def work(case):
    plen, G, L = _sizes(case)
    N, T = sum(G), case["max_new"]
    if case["kind"] == "scores":
        tokens = sum(L)
        return {"bytes": 8 * tokens + 16 * N + 24 * len(G), "flops": 8 * tokens}
    s = _shape(case)
    eb = 4 if s.dtype == "f32" else 2
    q, kv = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    layer = s.d_model * (q + 2 * kv) + q * s.d_model + 3 * s.d_model * s.ffn_dim
    lm, kvb = s.vocab * s.d_model, s.n_layers * 2 * kv * eb
    pre = sum(plen)
    att = 4 * q * s.n_layers                       # flops per (query, key)
    weights = (s.n_layers * layer + lm) * eb
    off = [g for g, n in enumerate(G) for _ in range(n)]
    rows = sum(L) - N                              # positions fed back through the decoder
    flops = 2 * (pre + rows) * s.n_layers * layer + 2 * (len(G) + rows) * lm
    flops += att * (sum(n * (n + 1) // 2 for n in plen) +
                    sum((n - 1) * plen[off[i]] + (n - 1) * n // 2 for i, n in enumerate(L)))
    byts = weights + (pre + rows) * kvb + 4 * (pre + 2 * N * T)
    if case["kind"] == "recompute":
        return {"bytes": byts, "flops": flops}
    for t in range(1, max(L)):                      # each decode step: the weights, every active group's prompt once, own keys and values
        act = [i for i, n in enumerate(L) if n > t]
        byts += weights + kvb * (sum(plen[g] for g in {off[i] for i in act}) + len(act) * t)
    return {"bytes": byts + 4 * case["dump"] * N * s.vocab, "flops": flops}


# ---------------------------------------------------------------- 64 bits
def exact(case, seed):
    if case["kind"] == "scores":
        return _exact_scores(case, seed)
    with torch.no_grad():
        return _exact_model(case, seed)


def _exact_model(case, seed):
    """The decoder in float64.  Keys and values are rounded to the cache's storage type (part of the model's
    definition); everything else is exact."""
    s = _shape(case)
    w = _weights(s, seed)
    prompts, G, L, tok = _token_inputs(case, seed)
    N, T, D = sum(G), case["max_new"], case["dump"]
    hd, nq, nkv, rep = s.head_dim, s.n_q_heads, s.n_kv_heads, s.n_q_heads // s.n_kv_heads
    inv = float(s.rope_theta) ** (-2.0 * torch.arange(hd // 2, device="cuda", dtype=torch.float64) / hd)
    kvt = torch.bfloat16 if s.dtype == "bf16" else torch.float32
    layers = [{k: t.double() for k, t in lw.items()} for lw in w.layers]
    head = w.lm_head.double()

    def norm(x):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + s.rms_eps)

    def stored(x):
        return x.float().to(kvt).double()

    def rope(x, pos):                               # x [..., n, heads, hd], pos [n]
        a = pos.double()[:, None] * inv
        c, sn = a.cos()[:, None, :], a.sin()[:, None, :]
        x1, x2 = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([x1 * c - x2 * sn, x2 * c + x1 * sn], -1)

    def forward(ids, pos0, cache):
        """ids [B, n] at positions pos0.. of B sequences behind a shared prefix (cache per layer: keys and values
        [nkv, L, hd], or None for a prompt).  Returns the final norm [B, n, d] and the new keys and values."""
        B, n = ids.shape
        pos = torch.arange(pos0, pos0 + n, device="cuda")
        hidden = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
        x = w.embed[ids.long()].double()
        kept = []
        for li, lw in enumerate(layers):
            h = norm(x)
            qh = rope((h @ lw["wq"].T).view(B, n, nq, hd), pos)
            k = stored(rope((h @ lw["wk"].T).view(B, n, nkv, hd), pos))
            v = stored((h @ lw["wv"].T).view(B, n, nkv, hd))
            kept.append((k, v))
            o = torch.empty(B, n, nq, hd, device="cuda", dtype=torch.float64)
            for b in range(B):
                for hh in range(nq):
                    g = hh // rep
                    qq = qh[b, :, hh] / math.sqrt(hd)
                    sc = (qq @ k[b, :, g].T).masked_fill_(hidden, -math.inf)
                    vv = v[b, :, g]
                    if cache is not None:
                        sc = torch.cat([qq @ cache[li][0][0, :, g].T, sc], 1)
                        vv = torch.cat([cache[li][1][0, :, g], vv])
                    o[b, :, hh] = torch.softmax(sc, -1) @ vv
            x = x + o.view(B, n, nq * hd) @ lw["wo"].T
            h = norm(x)
            x = x + (torch.nn.functional.silu(h @ lw["w_gate"].T) * (h @ lw["w_up"].T)) @ lw["w_down"].T
        return norm(x), kept

    lp = torch.zeros(N, T, device="cuda", dtype=torch.float64)
    dump = torch.zeros(D, N, s.vocab, device="cuda", dtype=torch.float64) if D else None
    off = 0
    for p, ids in enumerate(prompts):
        g, n = G[p], int(L[off:off + G[p]].max())
        hp, cache = forward(ids[None], 0, None)
        h = hp[:, -1:].expand(g, 1, s.d_model)
        if n > 1:
            h = torch.cat([h, forward(tok[off:off + g, :n - 1], ids.numel(), cache)[0]], 1)
        for j in range(g):
            for t0 in range(0, int(L[off + j]), 1024):
                t1 = min(int(L[off + j]), t0 + 1024)
                z = h[j, t0:t1] @ head.T
                if t0 < D:
                    dump[t0:min(t1, D), off + j] = z[:min(t1, D) - t0]
                z = z / float(np.float32(case["temperature"]))
                y = tok[off + j, t0:t1].long()
                lp[off + j, t0:t1] = z.gather(1, y[:, None])[:, 0] - torch.logsumexp(z, -1)
        off += g
    if case["kind"] == "recompute":
        return {"lp": lp}
    return {"tokens": None, "lengths": torch.from_numpy(L).cuda(), "lp": lp, "logits": dump}


def _exact_scores(case, seed):
    st = _prepare_scores(case, seed)
    r, L = st["rewards"].double().cpu().numpy(), st["len"].cpu().numpy()
    new, old = st["new"].double().cpu().numpy(), st["old"].double().cpu().numpy()
    G = st["G"].cpu().numpy()
    N, T = new.shape
    adv, stats, keep, o = np.zeros(N), np.zeros((len(G), 4)), np.zeros(len(G), np.int32), 0
    for p, g in enumerate(G):
        x, ln = r[o:o + g], L[o:o + g]
        keep[p] = bool((x != x[0]).any())
        if keep[p]:
            adv[o:o + g] = (x - x.mean()) / (x.std(ddof=1) + float(np.float32(1e-6)))
        med = float(np.median(ln))
        stats[p] = [ln.max(), med, ln.max() / med, ln.max() / med > 1.25]
        o += g
    kept = np.full(len(G), -1, np.int32)
    ids = np.flatnonzero(keep)
    kept[:len(ids)] = ids
    use = np.repeat(keep, G).astype(bool)
    valid = (np.arange(T)[None, :] < L[:, None]) & use[:, None]
    rho = np.exp(np.where(valid, new - old, 0.0))
    a32 = adv.astype(np.float32).astype(np.float64)[:, None]
    t1, t2 = rho * a32, np.clip(rho, 0.8, 1.28) * a32
    term = np.where(valid, np.minimum(t1, t2), 0.0)
    n_tok, n_seq = int(valid.sum()), int(use.sum())
    if n_tok == 0:
        loss = np.zeros(4)
    else:
        agg = term.sum() / n_tok if case["mode"] == "token" else (term.sum(1) / L)[use].mean()
        loss = np.array([-agg, float((valid & (t2 < t1)).sum()) / n_tok, n_tok, n_seq])
    return {"adv": adv, "keep": keep, "kept": kept, "n": np.array([len(ids)], np.int32), "stats": stats, "loss": loss}
