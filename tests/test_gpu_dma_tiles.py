"""Direct-to-LDS projection tiles (more than 1024 rows: 128 rows x 128 to 320
columns, K steps of 64 through two LDS buffers) against the oracle at their
edges: row counts one over and one short of a tile, K of one step (64), two and
many, with and without a K split, widths that end inside a column tile, and
every epilogue (QKV + RoPE + KV append, SwiGLU, residual, the lm head's partial
logsumexps and predicted-token logits, at temperatures 1 and 0.7).

Tolerance: activations carry 2^-17 relative in hi + lo planes and sums are
fp32, so what shows is a key or value rounding the other way into the bf16
cache (2^-8 of that element): about 1e-3 in a log-probability, bound 4e-3.
"""
import numpy as np
import pytest

from oracle.grpo import teacher_forced_logprobs
from workload import ModelShape, make_weights
from rg_helpers import make_policy, oracle_for, prompts_to_device

pytestmark = pytest.mark.gpu

SHAPES = [ModelShape(2, 64, 1, 1, 64, 64, 144, 1e4, dtype="bf16"),        # K = 64: one step
          ModelShape(2, 128, 6, 2, 64, 320, 1040, 1e4, dtype="bf16"),     # K = 128, 384, 320
          ModelShape(1, 512, 4, 1, 128, 1344, 2064, 1e4, dtype="bf16")]   # K split two to five ways


@pytest.mark.timeout(300)
@pytest.mark.parametrize("si", range(len(SHAPES)))
@pytest.mark.parametrize("rows", [1025, 1151, 1152, 1153])
def test_dma_tiles_match_oracle(si, rows):
    import torch
    assert torch.cuda.is_available()
    shape = SHAPES[si]
    w = make_weights(shape, 4)
    rng = np.random.default_rng(rows + si)
    P = 8
    plens = np.full(P, rows // P)
    plens[-1] += rows - plens.sum()
    prompts = [rng.integers(0, shape.vocab - 1, size=int(n)).astype(np.int32) for n in plens]
    G = [1] * P
    # completions whose fed-back positions number `rows` in one chunk
    lengths = (plens + 1).astype(np.int32)
    max_new = int(lengths.max())
    tok = rng.integers(0, shape.vocab - 1, size=(P, max_new)).astype(np.int32)
    pol = make_policy(shape, w, max_seqs=P, max_prompts=P, max_prompt_tokens=rows, max_context=int(plens.max()) + max_new)
    print(f"dma tiles: shape {si}, {rows} rows", flush=True)
    T = 0.7 if rows == 1152 else 1.0
    got = pol.recompute_logprobs(prompts_to_device(prompts), G, torch.from_numpy(tok).cuda(),
                                 torch.from_numpy(lengths).cuda(), temperature=T).cpu().numpy()
    want = teacher_forced_logprobs(oracle_for(shape, w), prompts, G, tok, lengths, temperature=T)
    valid = np.arange(max_new)[None, :] < lengths[:, None]
    gap = float(np.max(np.abs(got[valid] - want[valid])))
    print(f"gap {gap:.2e}", flush=True)
    assert np.isfinite(got).all() and gap <= 4e-3
    pol.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("dtype,hd", [("bf16", 64), ("f32", 32)])
def test_recompute_across_chunks(dtype, hd):
    """More completion positions than a recompute chunk holds (at most 4096 rows):
    a sequence split over the boundary attends to its own earlier positions from
    the first chunk and scores like any other.  The prompts alone (60 tokens)
    do not bound the chunk.  Tolerance as above; fp32 models 5e-5."""
    import torch
    assert torch.cuda.is_available()
    shape = ModelShape(2, 64, 2, 1, hd, 128, 144, 1e4, dtype=dtype)
    w = make_weights(shape, 6)
    rng = np.random.default_rng(11)
    P, G, max_new = 3, [9, 8, 8], 190
    N = sum(G)
    prompts = [rng.integers(0, shape.vocab - 1, size=20).astype(np.int32) for _ in range(P)]
    lengths = rng.integers(160, max_new + 1, size=N).astype(np.int32)
    rows = int(lengths.sum()) - N
    starts = np.concatenate([[0], np.cumsum(lengths - 1)])
    assert 4096 < rows and 4096 not in starts          # the boundary falls inside a sequence
    tok = rng.integers(0, shape.vocab - 1, size=(N, max_new)).astype(np.int32)
    print(f"recompute chunks: {dtype}, {rows} rows", flush=True)
    pol = make_policy(shape, w, max_seqs=N, max_prompts=P, max_prompt_tokens=60, max_context=20 + max_new)
    got = pol.recompute_logprobs(prompts_to_device(prompts), G, torch.from_numpy(tok).cuda(),
                                 torch.from_numpy(lengths).cuda()).cpu().numpy()
    want = teacher_forced_logprobs(oracle_for(shape, w), prompts, G, tok, lengths)
    valid = np.arange(max_new)[None, :] < lengths[:, None]
    gap = float(np.max(np.abs(got[valid] - want[valid])))
    print(f"gap {gap:.2e}", flush=True)
    assert np.isfinite(got).all() and gap <= (5e-5 if dtype == "f32" else 4e-3)
    pol.close()


@pytest.mark.timeout(300)
def test_lm_head_in_passes():
    """A chunk of more rows (5003: as many as prompt tokens) than the lm head
    scores in one pass (4096 at 16 tokens of vocabulary): the rows of the second
    pass take their own norm factors, targets and outputs.  Tolerance as above."""
    import torch
    assert torch.cuda.is_available()
    shape = ModelShape(1, 64, 1, 1, 64, 64, 16, 1e4, rms_eps=1e-6, dtype="bf16")
    w = make_weights(shape, 12)
    rng = np.random.default_rng(13)
    w.final_norm[:] = rng.uniform(1.0, 5.0, shape.d_model)   # values apart, so that another row's would show
    P = 25
    plens = np.full(P, 200)
    plens[-1] = 203
    prompts = [rng.integers(0, shape.vocab - 1, size=int(n)).astype(np.int32) for n in plens]
    lengths = (plens + 1).astype(np.int32)
    max_new = int(lengths.max())
    tok = rng.integers(0, shape.vocab - 1, size=(P, max_new)).astype(np.int32)
    print(f"lm head in passes: {plens.sum()} rows", flush=True)
    pol = make_policy(shape, w, max_seqs=P, max_prompts=P, max_prompt_tokens=int(plens.sum()), max_context=max_new + 203)
    got = pol.recompute_logprobs(prompts_to_device(prompts), [1] * P, torch.from_numpy(tok).cuda(),
                                 torch.from_numpy(lengths).cuda(), temperature=0.7, profile=True).cpu().numpy()
    assert pol.kernel_times(1)["gemm_lm"][1] == 2            # passes over the one chunk
    want = teacher_forced_logprobs(oracle_for(shape, w), prompts, [1] * P, tok, lengths, temperature=0.7)
    valid = np.arange(max_new)[None, :] < lengths[:, None]
    gap, spread = float(np.max(np.abs(got[valid] - want[valid]))), float(want[valid].std())
    print(f"gap {gap:.2e}, spread of the values {spread:.2f}", flush=True)
    assert np.isfinite(got).all() and gap <= 4e-3 < spread / 50
    pol.close()
