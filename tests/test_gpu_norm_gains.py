"""RMSNorm folded into the projections around it (operand x * gain, products
scaled by the row's 1 / rms from per-tile partial sums of squares) with gains
that are not 1 and an epsilon that matters, on every route that hands partial
sums over: split-K reductions (few rows), unsplit tiles, the direct-to-LDS tiles
(more than 1024 rows), fp32 tiles, and the lm head of rollout and recompute.
Teacher-forced rollout logits and recomputed log-probabilities against the
oracle.  Tolerances: fp32 sums 5e-5 for fp32 models (logits of order 3); bf16
models as everywhere, 1e-2 and 2e-2.
"""
import numpy as np
import pytest

from oracle.grpo import teacher_forced_logprobs
from oracle.rollout import rollout as oracle_rollout
from workload import ModelShape, make_weights
from rg_helpers import make_policy, oracle_for, prompts_to_device

pytestmark = pytest.mark.gpu

CASES = [("f32", 3, 40, 6), ("bf16", 3, 40, 6), ("bf16", 6, 230, 5), ("f32", 5, 60, 40)]   # dtype, prompts, length, max_new


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dtype,P,plen,max_new", CASES)
@pytest.mark.parametrize("d", [256, 1088])
def test_gains_and_epsilon(dtype, P, plen, max_new, d):
    import torch
    assert torch.cuda.is_available()
    shape = ModelShape(2, d, 4, 2, 64, 704, 528, 1e4, rms_eps=0.05, dtype=dtype)
    w = make_weights(shape, 8)
    rng = np.random.default_rng(d + P)
    for lw in w.layers:
        for n in ("attn_norm", "ffn_norm"):
            lw[n] = (rng.uniform(0.2, 2.0, d) * rng.choice([-1, 1], d)).astype(np.float32)
    w.final_norm[:] = rng.uniform(0.2, 2.0, d)
    G = [1 + p % 3 for p in range(P)]
    N = sum(G)
    prompts = [rng.integers(0, shape.vocab - 1, size=plen + p).astype(np.int32) for p in range(P)]
    L = rng.integers(1, max_new + 1, size=N).astype(np.int32)
    L[0] = max_new
    print(f"norm gains: {dtype}, d {d}, {P} prompts of {plen}.., {N} sequences, lengths {L.tolist()}", flush=True)
    model = oracle_for(shape, w)
    ref = oracle_rollout(model, prompts, G, max_new, 3, L, record_steps=max_new)
    pol = make_policy(shape, w, max_seqs=N, max_prompts=P, max_prompt_tokens=sum(len(p) for p in prompts),
                      max_context=plen + P + max_new)
    ft, dp = torch.from_numpy(ref["tokens"]).cuda(), prompts_to_device(prompts)
    _, ln, lp, dump = pol.rollout(dp, G, max_new, 3, forced_len=L, force_tokens=ft, dump_steps=max_new)
    dump, lp = dump.cpu().numpy(), lp.cpu().numpy()
    np.testing.assert_array_equal(ln.cpu().numpy(), L)
    gap = max(float(np.max(np.abs(dump[t, s] - ref["logits"][(s, t)]))) for s in range(N) for t in range(int(L[s])))
    want = teacher_forced_logprobs(model, prompts, G, ref["tokens"], ref["lengths"])
    got = pol.recompute_logprobs(dp, G, ft, torch.from_numpy(ref["lengths"]).cuda()).cpu().numpy()
    valid = np.arange(max_new)[None, :] < L[:, None]
    lgap = float(np.max(np.abs(got[valid] - want[valid])))
    print(f"logit gap {gap:.2e}, recompute gap {lgap:.2e}", flush=True)
    assert gap <= (5e-5 if dtype == "f32" else 1e-2) and lgap <= (5e-5 if dtype == "f32" else 2e-2)
    pol.close()
