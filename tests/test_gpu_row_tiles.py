"""Row-tile attention (prompt prefill and recompute rows of bf16 models: up to
128 query rows, positions x GQA heads, per workgroup, 32 per wave) against the
row-by-row pass, which shares neither its staging nor its softmax code, at the
edges of its tiles: tiles of 128 / rep positions, one short, full and one over;
32-token context blocks with remainders; 1 to 8 query heads per kv head, kv
heads that divide the 8 XCDs and that do not; both head sizes.

Tolerance.  Both passes carry q and p as hi + lo bf16 planes (2^-17 relative),
so with one layer (no attention output reaches a cache) log-probabilities of
order 10 from logits of order 1 agree to a few times 2^-17: 1e-4.  With two
layers an attention output that differs in its last bits can round a key or
value of the second layer the other way into the bf16 cache (2^-8 of that
element), which moves a log-probability by about 1e-3 at worst: 4e-3.
"""
import numpy as np
import pytest

from workload import ModelShape, make_weights
from rg_helpers import make_policy, prompts_to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,tol", [(1, 1e-4), (2, 4e-3)])
@pytest.mark.parametrize("n_q,n_kv,hd", [(2, 2, 64), (12, 2, 128), (7, 1, 128), (8, 1, 64), (6, 3, 64)])
def test_row_tiles_match_row_pass(n_q, n_kv, hd, layers, tol):
    import torch
    assert torch.cuda.is_available()
    shape = ModelShape(layers, 256, n_q, n_kv, hd, 512, 512, 1e4, dtype="bf16")
    tile = 128 // (n_q // n_kv)
    rng = np.random.default_rng(n_q * 10 + hd)
    plens = [tile - 1, tile, tile + 1, 1, 31, 32, 33, 2 * tile + 5, 300]
    prompts = [rng.integers(0, shape.vocab - 1, size=n).astype(np.int32) for n in plens]
    G = [1 + i % 2 for i in range(len(plens))]
    N, max_new = sum(G), tile + 3
    lengths = rng.integers(1, max_new + 1, size=N).astype(np.int32)
    lengths[:4] = [1, 2, tile + 1, max_new]     # no rows, one row, a full tile, one over (and the token before)
    tok = rng.integers(0, shape.vocab - 1, size=(N, max_new)).astype(np.int32)
    pol = make_policy(shape, make_weights(shape, 3), max_seqs=N, max_prompts=len(plens), max_prompt_tokens=sum(plens),
                      max_context=max(plens) + max_new)
    print(f"row tiles: {n_q}/{n_kv} heads of {hd}, {layers} layers, prompts {plens}, lengths {lengths.tolist()}",
          flush=True)
    dp, dt, dl = prompts_to_device(prompts), torch.from_numpy(tok).cuda(), torch.from_numpy(lengths).cuda()
    got = pol.recompute_logprobs(dp, G, dt, dl).cpu().numpy()
    want = pol.recompute_logprobs(dp, G, dt, dl, row_tiles=False).cpu().numpy()
    valid = np.arange(max_new)[None, :] < lengths[:, None]
    assert np.isfinite(got).all() and np.all(got[~valid] == 0)
    gap = float(np.max(np.abs(got[valid] - want[valid])))
    print(f"gap {gap:.2e}", flush=True)
    assert gap <= tol
    pol.close()
