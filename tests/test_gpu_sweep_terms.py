"""Efficiency sweep where its shortcuts can go wrong: tasks and attention series that change sides of the roofline among
the samples, next to ones that never do, for sample counts around the groups of eight, against the oracle."""
import numpy as np
import pytest

from paper_2412_04788_amd import guide, workloads as wl
from tests import bridge

pytestmark = pytest.mark.gpu
TOL = 1e-9


def _check(ora, g, e_c, e_b, first, count, tm):
    import torch
    n = count
    out = {k: torch.full((n,), 7, dtype={"b_max": torch.int32, "feasible": torch.uint8}.get(k, torch.float64), device="cuda")
           for k in guide.STATS_COLUMNS}
    bridge.gpu_context(g).eval_grid(bridge.gpu_grid(g), first, n, stats=out, e_c=e_c, e_b=e_b, time_model=tm)
    torch.cuda.synchronize()
    exp = ora.eval_sweep_grid(bridge.ora_grid(g), e_c, e_b, first, n, time_model=tm)
    for k in guide.STATS_COLUMNS:
        got = bridge.to_np(out[k], np.uint32 if k == "b_max" else None)
        if got.dtype == np.float64:
            assert bridge.rel_err(got, exp[k]).max() <= TOL, k
        else:
            np.testing.assert_array_equal(got, exp[k])


# peak / bandwidth from 1.25 (attention of a decode step is compute bound) over the point where a decode step's
# series changes sides inside a generation to 5000 (the segments of a long prompt change sides)
RATIOS = [1.25, 7.9, 8.05, 60.0, 300.0, 2500.0, 5000.0]


@pytest.mark.parametrize("spread", [0.0, 0.1, 1.5])
@pytest.mark.parametrize("n_eff", [2, 7, 8, 9, 33, 64])
def test_terms_that_change_sides(ora, n_eff, spread):
    hws = [wl.Hardware(r * 2e12, 2e12, 200 * wl.GIB, 1.6e11, 1e-6) for r in RATIOS]
    g = wl.make_grid([wl.DENSE_7B, wl.DENSE_70B, wl.MOE_8X], hws, wl.Axis.table([1, 3, 200]), wl.Axis.table([50, 3000, 20000]),
                     wl.Axis.table([1, 2, 900]), wl.Axis.table([1, 8]), wl.Axis.table([16, 4]), wl.Axis.table([16, 32]),
                     wl.Axis.table([1000, 2048, 8192]))
    rng = np.random.default_rng(n_eff)
    e_c, e_b = np.exp(spread * rng.standard_normal((2, n_eff)))
    _check(ora, g, e_c, e_b, 0, 2048, 0)
    _check(ora, g, e_c, e_b, g.size // 3 + 1, 2001, 0)
    _check(ora, g, e_c, e_b, g.size - 1500, 1500, 0)
    _check(ora, g, e_c, e_b, 7, 500, 1)


def test_many_coefficient_rows_and_extreme_samples(ora):
    g = wl.make_grid([wl.DENSE_7B, wl.DENSE_13B, wl.DENSE_34B, wl.DENSE_70B, wl.MOE_8X], wl.hw_profiles(4, 1), wl.Axis.table([5]),
                     wl.Axis.table([300, 9000]), wl.Axis.table([40]), wl.Axis.table([1, 2, 3, 4, 5, 6, 8]),
                     wl.Axis.table([16, 8, 4]), wl.Axis.table([16]), wl.Axis.table([2048]))
    e_c, e_b = wl.efficiency_pairs(n=16)
    _check(ora, g, e_c, e_b, 0, g.size, 0)
    e_c, e_b = e_c.copy(), e_b.copy()
    e_c[3], e_b[3], e_c[5], e_b[5] = 1e-150, 1e150, 1e120, 1e-120
    _check(ora, g, e_c, e_b, 0, g.size, 0)


def test_subnormal_efficiencies_come_last(ora):
    """A sample whose reciprocal overflows is the slowest of all, not no number: percentiles of the others are what they
    are without it.  (Its own time, and a mean that holds it, overflow or are beyond 1e280.)"""
    g = wl.make_grid([wl.DENSE_7B, wl.MOE_8X], [wl.Hardware(3e14, 2e12, 200 * wl.GIB, 1.6e11, 1e-6), wl.HW_TINY],
                     wl.Axis.table([1, 3, 200]), wl.Axis.table([50, 20000]), wl.Axis.table([1, 2, 300]), wl.Axis.table([1, 8]),
                     wl.Axis.table([16]), wl.Axis.table([16]), wl.Axis.table([2048]))
    import torch
    e_c, e_b = wl.efficiency_pairs(n=24)
    for tiny_c, tiny_b in ((5e-324, 1.0), (1.0, 1e-310), (1e-309, 1e-309)):
        c, b = e_c.copy(), e_b.copy()
        c[5], b[5] = tiny_c, tiny_b
        out = {k: torch.zeros(g.size, dtype={"b_max": torch.int32, "feasible": torch.uint8}.get(k, torch.float64), device="cuda")
               for k in guide.STATS_COLUMNS}
        bridge.gpu_context(g).eval_grid(bridge.gpu_grid(g), 0, g.size, stats=out, e_c=c, e_b=b)
        torch.cuda.synchronize()
        # the sample is replaced by one that is slow as well, but within the range
        c[5], b[5] = max(tiny_c, 1e-20), max(tiny_b, 1e-20)
        exp = ora.eval_sweep_grid(bridge.ora_grid(g), c, b, 0, g.size)
        for k in ("ttft_p10", "ttft_p90", "t_batch_p10", "t_batch_p90"):
            assert bridge.rel_err(bridge.to_np(out[k]), exp[k]).max() <= TOL, (k, tiny_c, tiny_b)
        for k in ("ttft_mean", "t_batch_mean"):
            assert (bridge.to_np(out[k]) > 1e280).all(), (k, tiny_c, tiny_b)
