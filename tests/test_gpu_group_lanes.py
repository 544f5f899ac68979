"""Group kernels (advantage, zero-variance filter, straggler statistics) where
their launch changes: 16, 32 or 64 lanes per group by the average size, one
tile of groups validated and placed by a single load up to 1024 groups and
tiles of 1024 beyond, one or four waves per group in the statistics.  Against
the oracle: advantages within 1e-5 relative (fp32 results of fp64 sums), the
filter and the statistics bit for bit, also with a NaN or an infinity among the
rewards; an invalid partition is refused on both paths."""
import numpy as np
import pytest

from oracle.advantage import group_advantage as oracle_adv, zero_variance_filter as oracle_filter
from oracle.sagc import group_stats as oracle_stats

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 63, 65, 1023, 1024, 1025])
@pytest.mark.parametrize("g", [1, 16, 17, 32, 33, 64, 65])
def test_group_kernels_at_launch_edges(P, g):
    import torch
    import paper_2606_02218_amd as rg
    rng = np.random.default_rng(P * 100 + g)
    G = np.full(P, g, np.int32)
    if P > 2:                                   # ragged around the same average
        G[0], G[1] = 1, 2 * g - 1
    N = int(G.sum())
    r = (rng.random(N) < rng.choice([0.0, 0.5, 1.0], size=P).repeat(G)).astype(np.float32)
    L = rng.integers(1, 5000, size=N).astype(np.int32)
    print(f"group launch edge: P {P}, G about {g}, N {N}", flush=True)
    Gd = torch.from_numpy(G).cuda()
    got = rg.group_advantage(torch.from_numpy(r).cuda(), Gd).cpu().numpy()
    np.testing.assert_allclose(got, oracle_adv(r, G, np.float32(1e-6)), rtol=1e-5, atol=1e-7)
    r[rng.integers(0, N)] = np.nan
    r[rng.integers(0, N)] = np.inf
    keep, kept, n = (t.cpu().numpy() for t in rg.group_filter(torch.from_numpy(r).cuda(), Gd))
    want_keep, want_ids = oracle_filter(r, G)
    np.testing.assert_array_equal(keep, want_keep)
    assert int(n[0]) == len(want_ids)
    np.testing.assert_array_equal(kept[:len(want_ids)], want_ids)
    st = rg.Sagc().group_stats(torch.from_numpy(L).cuda(), Gd).cpu().numpy()
    np.testing.assert_array_equal(st, np.asarray(oracle_stats(L, G, 1.25), np.float32))
    G[-1] += 1                                   # a partition that does not add up
    Gd = torch.from_numpy(G).cuda()
    assert np.isnan(rg.group_advantage(torch.from_numpy(r).cuda(), Gd).cpu().numpy()).all()
    assert int(rg.group_filter(torch.from_numpy(r).cuda(), Gd)[2].cpu()[0]) == -1


@pytest.mark.parametrize("P", [2, 7, 64, 300, 1024, 1500])
@pytest.mark.parametrize("g", [1, 4, 20])
@pytest.mark.parametrize("big", [64, 65, 128, 129, 1024])
def test_large_groups_among_small_ones(P, g, big):
    """The lanes of a group follow the average size; in the advantage one that
    takes more than four rounds of them is left to a whole wave, in the filter
    (a lane per group from some 64 groups on) one alike through its first 128.
    Large groups at either end and side by side in one wave's turn, some of them
    constant, and one with a NaN."""
    import torch
    import paper_2606_02218_amd as rg
    rng = np.random.default_rng(P * 10000 + g * 1000 + big)
    G = rng.integers(1, g + 1, size=P).astype(np.int32)
    at = sorted({0, P - 1, *range(P // 2, min(P, P // 2 + 3))})
    G[at] = big - np.arange(len(at)) % 2
    N, o = int(G.sum()), np.concatenate([[0], np.cumsum(G)])
    r = (rng.random(N) < rng.choice([0.0, 0.5, 1.0], size=P).repeat(G)).astype(np.float32)
    r[o[at[-1]]:o[at[-1] + 1]] = 0.25            # a large constant group, but for its last member
    r[o[at[-1] + 1] - 1] = 0.75
    print(f"skewed groups: P {P}, G up to {g}, {len(at)} of {big}, N {N}", flush=True)
    Gd = torch.from_numpy(G).cuda()
    got = rg.group_advantage(torch.from_numpy(r).cuda(), Gd).cpu().numpy()
    np.testing.assert_allclose(got, oracle_adv(r, G, np.float32(1e-6)), rtol=1e-5, atol=1e-7)
    r[o[at[0]]] = np.nan
    keep, kept, n = (t.cpu().numpy() for t in rg.group_filter(torch.from_numpy(r).cuda(), Gd))
    want_keep, want_ids = oracle_filter(r, G)
    np.testing.assert_array_equal(keep, want_keep)
    assert int(n[0]) == len(want_ids)
    np.testing.assert_array_equal(kept[:len(want_ids)], want_ids)
    L = rng.integers(1, 50, size=N).astype(np.int32)
    st = rg.Sagc().group_stats(torch.from_numpy(L).cuda(), Gd).cpu().numpy()
    np.testing.assert_array_equal(st, np.asarray(oracle_stats(L, G, 1.25), np.float32))


@pytest.mark.timeout(120)
def test_statistics_of_more_groups_than_one_row_of_blocks():
    """2^20 groups and one more: blocks come in rows of 2^20.  The last groups
    of both rows and some between, against numpy."""
    import torch
    import paper_2606_02218_amd as rg
    P = (1 << 20) + 1
    rng = np.random.default_rng(8)
    L = rng.integers(1, 5000, size=(P, 2)).astype(np.int32)
    print(f"statistics of {P} groups", flush=True)
    st = rg.Sagc().group_stats(torch.from_numpy(L.reshape(-1)).cuda(),
                               torch.full((P,), 2, dtype=torch.int32, device="cuda")).cpu().numpy()
    lmax, med = L.max(1).astype(np.float64), L.sum(1) / 2.0
    want = np.stack([lmax, med, lmax / med, (lmax / med > 1.25)], 1).astype(np.float32)
    np.testing.assert_array_equal(st, want)
