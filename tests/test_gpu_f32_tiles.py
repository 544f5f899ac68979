"""fp32 models' projections (16- and 64-row tiles of fp32 MFMAs, K shared by
four waves, fused epilogues) and attention (token groups in LDS, direct output
of a single chunk) against the float64 oracle at the edges of their tiles:
row counts around 16 and 64 and around the switch to 64-row tiles (129 rows
with 2048 gate/up columns), a vocabulary that ends in half a column tile, a
K of one turn (64) and 32 to 512 attention outputs per kv head.

Tolerance: every value is fp32 (2^-24 relative per operation); sums of at most
1024 terms through two layers and logits of order 1 leave a few times 1e-6.
The bound is 2e-5.
"""
import numpy as np
import pytest

from workload import ModelShape, make_weights
from rg_helpers import make_policy, oracle_for, prompts_to_device

pytestmark = pytest.mark.gpu

SHAPES = [ModelShape(2, 64, 2, 2, 32, 128, 48, 1e4, dtype="f32"),
          ModelShape(2, 256, 6, 2, 64, 1024, 528, 1e4, dtype="f32"),
          ModelShape(1, 128, 8, 2, 128, 256, 80, 1e4, dtype="f32")]


@pytest.mark.parametrize("si", range(len(SHAPES)))
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 64, 65, 128, 129, 193, 300])
def test_f32_prefill_logits(si, rows):
    import torch
    assert torch.cuda.is_available()
    shape = SHAPES[si]
    w = make_weights(shape, 2)
    rng = np.random.default_rng(rows)
    cut = rows // 3
    prompts = [rng.integers(0, shape.vocab - 1, size=n).astype(np.int32) for n in (cut, rows - cut) if n]
    pol = make_policy(shape, w, max_seqs=len(prompts), max_prompts=len(prompts), max_prompt_tokens=rows,
                      max_context=rows + 1)
    print(f"f32 tiles: shape {si}, {rows} rows", flush=True)
    _, _, _, dump = pol.rollout(prompts_to_device(prompts), [1] * len(prompts), 1, 7, dump_steps=1)
    dump = dump.cpu().numpy()
    model = oracle_for(shape, w)
    for p, ids in enumerate(prompts):
        want = model.forward(ids, np.arange(len(ids)), model.new_cache())[-1]
        assert float(np.max(np.abs(dump[0, p] - want))) <= 2e-5
    pol.close()
