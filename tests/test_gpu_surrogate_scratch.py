"""grpo_surrogate_scratch (per-sequence records in the caller's memory) equals
grpo_surrogate bit for bit inside 16 N bytes, refuses a missing or misaligned
scratch on the host, and the binding gives the same result on the current stream
(scratch from torch's allocator), and on a given stream."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,T,mode", [(1, 1, "token"), (5, 255, "seq"), (64, 1025, "token"), (700, 9, "seq")])
def test_scratch_surrogate_equals_the_allocating_one(N, T, mode):
    import torch
    import paper_2606_02218_amd as rg
    from paper_2606_02218_amd import _lib
    lib = rg.load_library()
    rng = np.random.default_rng(N + T)
    L = rng.integers(1, T + 1, size=N).astype(np.int32)
    old = rng.normal(-3.0, 1.0, (N, T)).astype(np.float32)
    new = (old + rng.normal(0, 0.2, (N, T))).astype(np.float32)
    d = [torch.from_numpy(a).cuda() for a in (new, old, rng.normal(size=N).astype(np.float32), L)]
    G = torch.tensor([N], dtype=torch.int32, device="cuda")
    want = torch.empty(4, dtype=torch.float64, device="cuda")
    print(f"surrogate scratch: N {N}, T {T}, {mode}", flush=True)
    a = [t.data_ptr() for t in d] + [G.data_ptr(), 1, N, T, 0, 0.2, 0.28, _lib.LOSS_MODES[mode], want.data_ptr()]
    assert lib.grpo_surrogate(*a, _lib._stream_ptr()) == _lib.RG_OK
    got = rg.grpo_surrogate(*d, G, eps_lo=0.2, eps_hi=0.28, mode=mode)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    other = rg.grpo_surrogate(*d, G, eps_lo=0.2, eps_hi=0.28, mode=mode, stream=side)
    torch.cuda.synchronize()
    w = want.cpu().numpy()
    assert np.array_equal(got.cpu().numpy(), w) and np.array_equal(other.cpu().numpy(), w)


@pytest.mark.parametrize("N,T,mode", [(1, 1, "seq"), (129, 300, "token"), (1000, 17, "seq")])
def test_scratch_surrogate_stays_in_its_scratch(N, T, mode):
    """The entry point itself, on 16 N bytes between guard words: equal to
    grpo_surrogate bit for bit, the records written, nothing beside them."""
    import torch
    import paper_2606_02218_amd as rg
    from paper_2606_02218_amd import _lib
    lib = rg.load_library()
    rng = np.random.default_rng(7 * N + T)
    L = rng.integers(1, T + 1, size=N).astype(np.int32)
    old = rng.normal(-3.0, 1.0, (N, T)).astype(np.float32)
    new = (old + rng.normal(0, 0.2, (N, T))).astype(np.float32)
    d = [torch.from_numpy(a).cuda() for a in (new, old, rng.normal(size=N).astype(np.float32), L)]
    G = torch.tensor([N], dtype=torch.int32, device="cuda")
    print(f"surrogate scratch with guards: N {N}, T {T}, {mode}", flush=True)
    out = [torch.empty(4, dtype=torch.float64, device="cuda") for _ in range(2)]
    guard, word = 64, 0x5A5A5A5A5A5A5A5A
    mem = torch.full((guard + 2 * N + guard,), word, dtype=torch.int64, device="cuda")
    args = [t.data_ptr() for t in d] + [G.data_ptr(), 1, N, T, 0, 0.2, 0.28, _lib.LOSS_MODES[mode]]
    assert lib.grpo_surrogate(*args, out[0].data_ptr(), _lib._stream_ptr()) == _lib.RG_OK
    rc = lib.grpo_surrogate_scratch(*args, out[1].data_ptr(), mem.data_ptr() + 8 * guard, _lib._stream_ptr())
    assert rc == _lib.RG_OK
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
    m = mem.cpu().numpy()
    assert (m[:guard] == word).all() and (m[-guard:] == word).all()
    assert (m[guard:-guard].reshape(N, 2) != word).all()


def test_scratch_surrogate_refuses_bad_scratch():
    import paper_2606_02218_amd as rg
    from paper_2606_02218_amd import _lib
    lib = rg.load_library()
    p = [C.c_void_p(256 * (i + 1)) for i in range(6)]
    for bad in (None, C.c_void_p(8)):
        rc = lib.grpo_surrogate_scratch(p[0], p[1], p[2], p[3], p[4], 1, 4, 8, None, 0.2, 0.2, 0, p[5], bad, None)
        assert rc == _lib.RG_EINVAL and b"scratch" in lib.rg_last_error()


@pytest.mark.timeout(120)
@pytest.mark.parametrize("N", [(1 << 20) + 1, (1 << 24) + 1])
def test_more_sequences_than_one_row_of_blocks(N):
    """2^24 sequences of one token and one more: with 256 threads each they pass
    the 2^32 threads that one dimension of a launch holds.  Terms of one sign, so
    that sums of 1.7e7 of them agree to a few fp64 roundings (1e-12)."""
    import torch
    import paper_2606_02218_amd as rg
    rng = np.random.default_rng(3)
    old = rng.normal(-3.0, 1.0, (N, 1)).astype(np.float32)
    new = (old + rng.normal(0, 0.2, (N, 1)).astype(np.float32)).astype(np.float32)
    adv = rng.uniform(0.1, 2.0, N).astype(np.float32)
    G = np.full(-(-N // 4096), 4096, np.int32)
    G[-1] = N - 4096 * (len(G) - 1)
    print(f"surrogate of {N} sequences", flush=True)
    d = [torch.from_numpy(a).cuda() for a in (new, old, adv, np.ones(N, np.int32), G)]
    got = rg.grpo_surrogate(*d, eps_lo=0.2, eps_hi=0.28, mode="token").cpu().numpy()
    rho = np.exp(new[:, 0].astype(np.float64) - old[:, 0])
    un, cl = rho * adv, np.clip(rho, 0.8, 1.28) * adv
    assert got[2] == N and got[3] == N
    assert got[0] == pytest.approx(-np.minimum(un, cl).mean(), rel=1e-12)
    assert got[1] == pytest.approx((cl < un).mean(), abs=3.0 / N)   # a clip decided by the last bit of exp
