"""Efficiency sweeps whose prefill columns are made by items of their own (many rows, six generation lengths and four
samples or more): the same bits as in pieces that are too small for that, whatever part of the grid is asked for; and the order in
which the samples are added up."""
import numpy as np
import pytest

from paper_2412_04788_amd import guide, workloads as wl
from tests import bridge

pytestmark = pytest.mark.gpu
PIECE = 60_000          # rows: fewer items than fill the chip


def _sweep(ctx, g, e_c, e_b, first, count, tm):
    import torch
    out = {k: torch.full((count + 2,), 7, dtype={"b_max": torch.int32, "feasible": torch.uint8}.get(k, torch.float64), device="cuda")
           for k in guide.STATS_COLUMNS}
    ctx.eval_grid(bridge.gpu_grid(g), first, count, stats={k: v[1:-1] for k, v in out.items() if k not in ("b_max", "feasible")} |
                  {k: out[k][:count] for k in ("b_max", "feasible")}, e_c=e_c, e_b=e_b, time_model=tm)
    torch.cuda.synchronize()
    res = {}
    for k, v in out.items():
        v = v.cpu().numpy()
        lo = 0 if k in ("b_max", "feasible") else 1
        assert (v[:lo] == 7).all() and (v[lo + count:] == 7).all(), k      # nothing beside the range
        res[k] = v[lo:lo + count]
    return res


# lengths of s_out, block sizes and token budgets; odd ranges of the grid; samples around a group of eight; coefficients in LDS or
# (99 rows) in lane
@pytest.mark.parametrize("n_so,n_blk,n_mbt,first,less,n_eff,tm,tp",
                         [(6, 1, 1, 0, 0, 9, 0, (1, 2, 8)), (8, 2, 3, 1237, 5, 8, 0, (1, 2, 8)), (7, 2, 5, 31, 40_001, 3, 1, (1, 2, 8)),
                          (64, 1, 2, 7, 0, 2, 0, (1, 2, 8)), (64, 1, 2, 7, 0, 4, 0, (1, 2, 8)), (7, 2, 5, 31, 40_001, 5, 1, (1, 2, 8)),
                          (6, 2, 2, 77, 9, 20, 0, range(1, 12)), (6, 2, 2, 77, 9, 20, 1, range(1, 12))])
def test_prefill_items(n_so, n_blk, n_mbt, first, less, n_eff, tm, tp):
    items_above = -(-170_000 // (n_so * n_mbt * 3 * len(tp)))              # settings of model, hw, batch, s_in
    n_b = -(-items_above // (3 * 2 * 3))
    g = wl.make_grid([wl.DENSE_7B, wl.DENSE_70B, wl.MOE_8X], wl.hw_profiles(5, 2),
                     wl.Axis.table([1 + 3 * i for i in range(min(n_b, 64))]),
                     wl.Axis.table([50, 3000, 20000] if n_b <= 64 else [50 + 399 * i for i in range(-(-items_above // (6 * 64)))]),
                     wl.Axis.table([1 + 13 * i for i in range(n_so)]), wl.Axis.table(list(tp)), wl.Axis.table([16, 8, 4]),
                     wl.Axis.table([16, 32][:n_blk]), wl.Axis.table([1000, 2048, 4096, 8192, 16384][:n_mbt]))
    count = g.size - first - less
    assert count // n_blk > 2 * 256 * 256                                  # more items than fill the chip
    e_c, e_b = wl.efficiency_pairs(n=n_eff)
    ctx = bridge.gpu_context(g)
    whole = _sweep(ctx, g, e_c, e_b, first, count, tm)
    for at in range(0, count, PIECE):
        n = min(PIECE, count - at)
        part = _sweep(ctx, g, e_c, e_b, first + at, n, tm)
        for k in guide.STATS_COLUMNS:
            np.testing.assert_array_equal(whole[k][at:at + n], part[k], err_msg=k)


def _added_up(times):
    """Sum over axis 0 in the documented order: groups of eight as trees, the rest one by one."""
    total, i, n = 0.0, 0, len(times)
    while i + 8 <= n:
        a = times[i:i + 8]
        total = total + (((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])))
        i += 8
    for t in times[i:]:
        total = total + t
    return total


# One GPU (no transfers) and samples that scale both rates by the same power of two: every time is the least one times a power
# of two, exactly, so the sums' roundings are known bit for bit.
@pytest.mark.parametrize("n_eff", [2, 7, 8, 9, 20, 64])
@pytest.mark.parametrize("tm", [0, 1])
def test_order_of_the_sums(n_eff, tm):
    g = wl.make_grid([wl.DENSE_7B, wl.MOE_8X], wl.hw_profiles(5, 2), wl.Axis.table([1, 7, 300]), wl.Axis.table([50, 3001]),
                     wl.Axis.table([1, 30, 1000]), wl.Axis.table([1]), wl.Axis.table([16, 4]), wl.Axis.table([16]), wl.Axis.table([1000, 8192]))
    power = (np.arange(n_eff) * 11) % 5                                   # 0 at first: sample 0 is among the fastest
    e = 0.5 ** power
    out = _sweep(bridge.gpu_context(g), g, e, e, 0, g.size, tm)
    # the least time is the p10: at least a tenth of the samples are as fast
    assert np.count_nonzero(power == 0) >= -(-n_eff // 10)
    for name in ("ttft", "t_batch"):
        times = out[name + "_p10"][None, :] * 2.0 ** power[:, None]
        np.testing.assert_array_equal(out[name + "_mean"], _added_up(times) / n_eff, err_msg=name)
    one_by_one = np.zeros(g.size)
    for t in out["t_batch_p10"][None, :] * 2.0 ** power[:, None]:
        one_by_one = one_by_one + t
    assert n_eff < 8 or (one_by_one != _added_up(times)).any()            # (the test can tell the orders apart)
