"""GPU parity: Philox blocks and sampling bits bit-exact; group advantage
within 1e-5 relative of the oracle; the zero-variance group filter bit-exact."""
import numpy as np
import pytest

from oracle.philox import philox4x64_10, gumbel_uniform_bits
from oracle.advantage import group_advantage as oracle_adv, zero_variance_filter
from workload import get_config, make_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rg():
    import torch
    assert torch.cuda.is_available()
    import paper_2606_02218_amd as rg
    return rg


def test_philox_blocks_bit_exact(rg):
    import torch
    rng = np.random.default_rng(0)
    ctr = rng.integers(0, 2 ** 63, size=(4096, 4), dtype=np.int64).view(np.uint64)
    ctr[:8] = np.array([[0, 0, 0, 0], [2 ** 64 - 1] * 4, [1, 2, 3, 4], [5, 0, 17, 0],
                        [18990, 4095, 511, 0], [0, 1, 0, 0], [7, 7, 7, 7], [2 ** 32, 2 ** 32 - 1, 9, 1]], np.uint64)
    for key in [(0, 0), (12345, 1), (2 ** 64 - 1, 2 ** 63 + 11)]:
        dev = torch.from_numpy(ctr.view(np.int64).copy()).cuda()
        out = rg.philox_blocks(key[0], key[1], dev).cpu().numpy().view(np.uint64)
        np.testing.assert_array_equal(out, philox4x64_10(ctr, key))


@pytest.mark.parametrize("seed,t,s,V", [(0, 0, 0, 512), (1234, 17, 63, 32000), (2 ** 63 + 5, 4095, 511, 151936),
                                        (7, 8191, 255, 152064)])
def test_gumbel_bits_bit_exact(rg, seed, t, s, V):
    got = rg.gumbel_bits(seed, t, s, V).cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(got, gumbel_uniform_bits(seed, t, s, V))


def test_gumbel_noise_over_every_uniform(rg):
    """The noise that the sampler adds, for each of the 2^23 uniforms its stream
    can give, against 64 bits.  A relative error of 2^-23 in the inner logarithm
    moves the noise by 1.2e-7; the outer one's value reaches 23.5 before the
    product with ln 2, whose last bit is 1.9e-6: 2e-6 in all, also in the tail
    near u = 1 that wins a draw, and 1e-7 rms (an ordinary value is below 4)."""
    import torch
    from paper_2606_02218_amd import _lib
    n = 1 << 23
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    print("Gumbel noise of 2^23 uniforms", flush=True)
    assert rg.load_library().rg_gumbel_noise(0, n, out.data_ptr(), _lib._stream_ptr()) == _lib.RG_OK
    u = (2.0 * np.arange(n) + 1.0) * 2.0 ** -24
    err = out.cpu().numpy().astype(np.float64) - (-np.log(-np.log(u)) + np.log(np.log(2.0)))
    print(f"max {np.abs(err).max():.3e}, rms {np.sqrt(np.mean(err * err)):.3e}", flush=True)
    assert np.abs(err).max() <= 2e-6 and np.sqrt(np.mean(err * err)) <= 1e-7
    part = torch.empty(1000, dtype=torch.float32, device="cuda")
    assert rg.load_library().rg_gumbel_noise(n - 1000, 1000, part.data_ptr(), _lib._stream_ptr()) == _lib.RG_OK
    assert torch.equal(part, out[-1000:])
    for first, m in ((-1, 4), (0, 0), (n - 3, 4)):
        assert rg.load_library().rg_gumbel_noise(first, m, out.data_ptr(), None) == _lib.RG_EINVAL


def _adv_case(rg, rewards, G, ddof=1):
    import torch
    r = torch.from_numpy(np.asarray(rewards, np.float32)).cuda()
    g = torch.from_numpy(np.asarray(G, np.int32)).cuda()
    got = rg.group_advantage(r, g, 1e-6, ddof).cpu().numpy()
    ref = oracle_adv(np.asarray(rewards, np.float32), G, np.float32(1e-6), ddof)
    np.testing.assert_allclose(got, ref, rtol=1e-5, atol=1e-7)
    return got


@pytest.mark.parametrize("ddof", [0, 1])
def test_advantage_layouts(rg, ddof):
    rng = np.random.default_rng(1)
    layouts = [[4] * 8, [16] * 32, list(make_inputs(get_config("1.5b-dyn"), 0).G), [1, 2, 3, 1000, 5],
               list(rng.integers(1, 9, size=3000)), [1]]
    for G in layouts:
        N = int(np.sum(G))
        _adv_case(rg, (rng.random(N) < 0.5).astype(np.float32), G, ddof)
        _adv_case(rg, rng.normal(size=N).astype(np.float32), G, ddof)


def test_advantage_constant_groups_and_invariants(rg):
    G = [4, 4, 8, 2]
    r = np.array([1, 1, 1, 1, 0, 0, 0, 0] + [1, 0, 0, 1, 1, 1, 0, 0] + [3, 3], np.float32)
    a = _adv_case(rg, r, G)
    assert np.all(a[:8] == 0) and np.all(a[-2:] == 0)
    seg = a[8:16].astype(np.float64)
    assert abs(seg.sum()) < 1e-6 * 8
    sd = np.std(r[8:16].astype(np.float64), ddof=1)
    assert abs(np.std(seg, ddof=1) - sd / (sd + 1e-6)) < 1e-6


def test_advantage_workload_rewards(rg):
    for name in ["tiny", "gpt2s", "1.5b", "1.5b-dyn", "7b"]:
        inp = make_inputs(get_config(name), 0)
        _adv_case(rg, inp.rewards, list(inp.G))


def test_advantage_bad_group_sizes_give_nan(rg):
    import torch
    r = torch.ones(8, device="cuda")
    for G in ([4, 3], [4, 0, 4], [4, 5], [2 ** 31 - 1, 2 ** 31 - 1, 10]):
        out = rg.group_advantage(r, torch.tensor(G, dtype=torch.int32, device="cuda")).cpu().numpy()
        assert np.all(np.isnan(out)), G


def _filter_case(rg, rewards, G):
    import torch
    r = torch.from_numpy(np.asarray(rewards, np.float32)).cuda()
    keep, ids, n = rg.group_filter(r, torch.from_numpy(np.asarray(G, np.int32)).cuda())
    ref_keep, ref_ids = zero_variance_filter(rewards, G)
    n = int(n.item())
    assert n == len(ref_ids)
    np.testing.assert_array_equal(keep.cpu().numpy(), ref_keep)
    ids = ids.cpu().numpy()
    np.testing.assert_array_equal(ids[:n], ref_ids)
    assert np.all(ids[n:] == -1)   # untouched past the kept count
    return ref_keep


def test_group_filter_layouts(rg):
    rng = np.random.default_rng(11)
    layouts = [[4] * 8, [16] * 32, list(make_inputs(get_config("1.5b-dyn"), 0).G), [1, 2, 3, 1000, 5],
               list(rng.integers(1, 9, size=3000)), [1], [2] * 2049]
    for G in layouts:
        N = int(np.sum(G))
        off = np.concatenate([[0], np.cumsum(G)])
        r = (rng.random(N) < rng.random()).astype(np.float32)
        _filter_case(rg, r, G)
        r = rng.normal(size=N).astype(np.float32)
        for p in range(0, len(G), 2):
            r[off[p]:off[p + 1]] = r[off[p]]
        keep = _filter_case(rg, r, G)
        assert keep[::2].sum() == 0


def test_group_filter_edge_values(rg):
    G = [2, 2, 2, 1, 2, 3]
    r = [0.0, -0.0, 1.0, float(np.nextafter(np.float32(1), np.float32(2))), np.nan, np.nan, np.nan, 5.0, 5.0,
         np.inf, np.inf, np.inf]
    _filter_case(rg, np.array(r, np.float32), G)
    _filter_case(rg, np.ones(64, np.float32), [64])
    _filter_case(rg, np.zeros(4096, np.float32), [1] * 4096)


def test_group_filter_workload_rewards(rg):
    for name in ["tiny", "gpt2s", "1.5b", "1.5b-dyn", "7b"]:
        inp = make_inputs(get_config(name), 0)
        _filter_case(rg, inp.rewards, list(inp.G))


def test_group_filter_bad_group_sizes(rg):
    import torch
    r = torch.ones(8, device="cuda")
    for G in ([4, 3], [4, 0, 4], [4, 5], [2 ** 31 - 1, 2 ** 31 - 1, 10]):
        keep, ids, n = rg.group_filter(r, torch.tensor(G, dtype=torch.int32, device="cuda"))
        assert int(n.item()) == -1, G
        assert np.all(ids.cpu().numpy() == -1), G


@pytest.mark.parametrize("n16,blocks", [(1, 1), (257, 3), (4096 * 33 + 5, 64), (1 << 20, 2048)])
def test_hbm_probe_copy_and_read(rg, n16, blocks):
    """The streaming ceiling probe (a measurement hook, not a path step):
    mode 1 copies every 16-byte piece, including the grid-stride tail;
    mode 0 stores, per thread, the xor of every word it read."""
    import torch
    g = torch.Generator().manual_seed(n16)
    src = torch.randint(-2 ** 31, 2 ** 31 - 1, (n16 * 4,), dtype=torch.int32, generator=g).cuda()
    dst = torch.zeros_like(src)
    rg.hbm_probe(src, dst, 1, blocks)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)
    sink = torch.zeros(blocks * 256, dtype=torch.int32, device="cuda")
    rg.hbm_probe(src, sink, 0, blocks)
    torch.cuda.synchronize()
    # thread i of the grid reads pieces i, i + T, i + 2T, ... (T = blocks * 256 threads)
    words = src.cpu().numpy().view(np.uint32).reshape(n16, 4)
    T = blocks * 256
    expect = np.zeros(T, np.uint32)
    for i in range(min(T, n16)):
        expect[i] = np.bitwise_xor.reduce(words[i::T].reshape(-1))
    np.testing.assert_array_equal(sink.cpu().numpy().view(np.uint32), expect)
