"""Pareto selections whose kept rows one block does not hold: row samples of either depth, parts with a few survivors, with
several rounds of them and with one bin too large for LDS, against the oracle (indices: exact)."""
import numpy as np
import pytest

from paper_2412_04788_amd import workloads as wl
from tests import bridge
from tests.test_gpu_select import _dev, _pareto

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    assert torch.cuda.is_available()
    return torch, bridge.gpu_context(wl.grid_tiny())


def _check(ora, setup, x, y, fe=None, cons=(), capacity=None):
    torch, ctx = setup
    got, m = _pareto(torch, ctx, _dev(torch, x), _dev(torch, y), None if fe is None else _dev(torch, fe),
                     [(_dev(torch, c), cap) for c, cap in cons], capacity)
    ok = np.ones(len(x), np.uint8) if fe is None else fe.copy()
    for c, cap in cons:
        ok &= (c <= cap).astype(np.uint8)
    exp = ora.pareto_sweep(x, y, ok)
    assert m == len(exp)
    np.testing.assert_array_equal(got, exp if capacity is None else exp[:capacity])
    return m


# one more than a block stages, the rows that a part's threads hold between its passes (10 240) and one more, the sample's depths
@pytest.mark.parametrize("n, kind", [(n, kind) for n in (4097, 10240, 10241, 16385, 65537) for kind in ("front", "triples", "near", "far")] +
                         [(400_000, "front"), (400_000, "triples"), (1_500_000, "near"), (1_500_001, "near")])
def test_fronts_by_size(ora, setup, n, kind):
    rng = np.random.default_rng(n)
    if kind == "front":                                 # every row: parts of n / 64 survivors, beyond 262 144 in rounds
        x = rng.permutation(n) + 1.0
        y = -x
    elif kind == "triples":                             # equal points in threes
        x = (rng.permutation(n) // 3) + 1.0
        y = 1.0 / x
    elif kind == "near":                                # a thin front before a cloud, ties in runs
        u = np.repeat(rng.random(n // 5 + 1), 5)[:n]
        x = np.exp(9.0 * u - 5.0)
        y = np.exp(2.0 - 4.0 * u + 0.4 * np.abs(np.repeat(rng.standard_normal(n // 5 + 1), 5)[:n]))
    else:                                               # most of x in a sliver of its range
        x = 1.0 + rng.random(n) ** 40
        y = 2.0 - x + 1e-3 * rng.random(n)
    _check(ora, setup, x, y)
    fe = (rng.random(n) < 0.7).astype(np.uint8)
    c, d = rng.random(n), rng.random(n)
    _check(ora, setup, x, y, fe, [(c, 0.8)])
    _check(ora, setup, x, y, fe, [(c, 0.8), (d, 0.9)], capacity=1000)


@pytest.mark.parametrize("n", [200_000, 1_600_000])
def test_survivors_of_one_bin_beyond_the_staging_arrays(ora, setup, n):
    rng = np.random.default_rng(n + 1)
    x, y = rng.random(n) * 100.0, rng.random(n) * 100.0
    odd = np.setdiff1d(np.arange(n), bridge.pareto_sample_rows(n))
    odd = rng.choice(odd, 12_000, replace=False)        # a staircase right of everything that is sampled
    x[odd] = 1000.0 + odd
    y[odd] = -1.0 * odd
    assert _check(ora, setup, x, y) > 8000


@pytest.mark.parametrize("n", [100_000, 1_600_000])
def test_no_sample_row_passes(ora, setup, n):
    rng = np.random.default_rng(n + 2)
    x, y = np.round(rng.random(n) * 1000.0, 1), np.round(rng.random(n) * 1000.0, 1)
    fe = np.ones(n, np.uint8)
    fe[bridge.pareto_sample_rows(n)] = 0
    _check(ora, setup, x, y, fe)
    _check(ora, setup, x, y, np.zeros(n, np.uint8))


def test_all_rows_in_one_bin_of_an_unsampled_range(ora, setup):
    # 13 600 kept rows that nothing prunes
    n = 30_000
    rng = np.random.default_rng(4)
    fe = np.ones(n, np.uint8)
    fe[bridge.pareto_sample_rows(n)] = 0
    x = np.round(rng.random(n) * 1000.0, 1)
    _check(ora, setup, x, 1e6 - 7.0 * x, fe)            # all of them on the front, many equal
    for x in (np.full(n, np.inf), np.full(n, -np.inf), np.round(rng.random(n), 3)):
        _check(ora, setup, x, np.round(rng.random(n) * 1000.0, 1), fe)


# one row, or several, far from all others, which the sample misses: the parts at the ends of x bin the others as without it
@pytest.mark.parametrize("n", [50_000, 200_000, 600_000, 1_900_800])
@pytest.mark.parametrize("far", ["right", "left", "both", "many"])
def test_far_rows(ora, setup, n, far):
    rng = np.random.default_rng(n + 3)
    x = rng.permutation(n) + 1.0
    y = -x
    odd = np.setdiff1d(np.arange(n), bridge.pareto_sample_rows(n))
    odd = rng.choice(odd, 2000 if far == "many" else 2, replace=False)
    if far in ("right", "both"):
        x[odd[0]], y[odd[0]] = (np.inf if n == 200_000 else 1e300), -1e9
    if far in ("left", "both"):
        x[odd[1]], y[odd[1]] = (-np.inf if n == 200_000 else 0.0), 1e9
    if far == "many":
        x[odd] = 1e300 * (1.0 + np.arange(2000.0))
        y[odd] = -1e9 - np.arange(2000.0)
    assert _check(ora, setup, x, y) == n


def _crowd(kind, n):
    """Rows that crowd in a few values of x, or at a few of its scales: one bin of any equal slicing holds most of them."""
    rng = np.random.default_rng(n)
    if kind == "one x":
        return np.full(n, 3.0), rng.random(n)
    if kind == "one x, few ys":                         # ties in y by the ten thousand, all on the front
        return np.full(n, -2.5), rng.integers(0, 7, n).astype(np.float64)
    if kind == "one point":
        return np.full(n, 1e-300), np.full(n, -np.inf)
    if kind == "few xs":
        x = rng.integers(1, 6, n).astype(np.float64)
        return x, np.round(rng.random(n), 4) - x
    if kind == "few points":                            # five of them, tied by the ten thousand, all on the front
        x = rng.integers(1, 6, n).astype(np.float64)
        return x, -x
    # clusters inside clusters inside clusters: slices of the widest range hold one, slices of its range one of its own
    rank = rng.permutation(n)
    same = rank // 3 if kind == "clusters, ties" else rank
    m = max(same.max() // 9, 1)
    outer = np.minimum(same // (3 * m), 2)
    x = np.ldexp(1.0, outer * 300 - 300) * (1.0 + np.ldexp(same // m - 3 * outer, -20) + np.ldexp(same % m, -51))
    return x, -1.0 * same


# a part's share beyond LDS, by far
@pytest.mark.parametrize("n", [4097, 9_001, 300_007, 1_600_000])
@pytest.mark.parametrize("kind", ["one x", "one x, few ys", "one point", "few xs", "few points", "clusters", "clusters, ties"])
def test_rows_that_crowd_in_x(ora, setup, kind, n):
    x, y = _crowd(kind, n)
    _check(ora, setup, x, y)
    fe = (np.random.default_rng(n + 1).random(n) < 0.5).astype(np.uint8)
    _check(ora, setup, x, y, fe, capacity=n // 3)
    _check(ora, setup, x, np.full(n, np.inf))


# records that one block stages: in a bin or two of their range, with and without ties
@pytest.mark.parametrize("n", [1024, 1025, 2047, 2048, 2049, 4095, 4096])
@pytest.mark.parametrize("kind", ["one x", "one x, few ys", "one point", "few xs", "few points", "clusters", "clusters, ties"])
def test_few_rows_that_crowd_in_x(ora, setup, kind, n):
    x, y = _crowd(kind, n)
    _check(ora, setup, x, y)
    x, y = x.copy(), y.copy()
    far = n // 2
    x[far], y[far] = np.inf, y.min() - 1.0              # the right end of the range far from all others
    _check(ora, setup, x, y)
    _check(ora, setup, np.append(x, 5.0)[1:], np.append(y, -np.inf)[1:])
    _check(ora, setup, x, np.full(n, np.inf))


@pytest.mark.parametrize("n, kind", [(4097, "one point"), (20_011, "clusters"), (300_007, "clusters, ties"), (300_007, "one point")])
def test_workspace_is_what_is_asked_for(setup, n, kind):
    torch, ctx = setup
    from paper_2412_04788_amd import guide
    x, y = (_dev(torch, a) for a in _crowd(kind, n))
    need = ctx.select_workspace_bytes(guide.SELECT_PARETO, n)
    buf = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    idx = torch.full((n,), -7, dtype=torch.int64, device="cuda")
    cnt = torch.full((1,), -7, dtype=torch.int64, device="cuda")
    with pytest.raises(guide.GuideError):
        ctx.select(guide.SELECT_PARETO, n, x, idx, None, cnt, buf[:need - 1], objective_y=y, capacity=n)
    ctx.select(guide.SELECT_PARETO, n, x, idx, None, cnt, buf[:need], objective_y=y, capacity=n)
    torch.cuda.synchronize()
    assert int(cnt[0]) == n and bool((idx >= 0).all())
    assert bool((buf[need:] == 0xA5).all())


def test_most_rows_end(setup):
    """2^32 - 4096 rows, all on the front: index arithmetic of the batched loops next to the end of 32 bits (a batch's end wraps)."""
    torch, ctx = setup
    from paper_2412_04788_amd import guide
    n = 2 ** 32 - 4096
    need = ctx.select_workspace_bytes(guide.SELECT_PARETO, n)
    if torch.cuda.mem_get_info()[0] < need + 16 * n + 2 ** 31:
        pytest.skip("200 GB of device memory")
    x = torch.arange(n, dtype=torch.float64, device="cuda")
    x += 2.0 ** 33                                      # one binade: the parts share the rows evenly
    y = -x
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    idx = torch.full((100_000,), -7, dtype=torch.int64, device="cuda")
    cnt = torch.full((1,), -7, dtype=torch.int64, device="cuda")
    ctx.select(guide.SELECT_PARETO, n, x, idx, None, cnt, ws, objective_y=y, capacity=idx.numel())
    torch.cuda.synchronize()
    assert int(cnt[0]) == n
    assert torch.equal(idx, torch.arange(idx.numel(), device="cuda"))
    del x, y, ws
    torch.cuda.empty_cache()


# members of a bin on either side of the line between pairwise tests and sorting, a third of them dominated, some equal
@pytest.mark.parametrize("n", [1024, 1025, 2048, 4096])
@pytest.mark.parametrize("members", [2, 63, 64, 65, 66, 512])
def test_members_of_a_bin(ora, setup, n, members):
    rank = np.random.default_rng(members).permutation(n)
    x = 1.0 + (rank // members) / (-(-n // members)) + (rank % members) * 2.0 ** -50
    _check(ora, setup, x, -1.0 * rank)
    _check(ora, setup, x, np.where(rank % 3 == 0, 1.0 - rank, -1.0 * (rank // 2)))
