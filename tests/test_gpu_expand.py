"""Kernels that expand runs of tiles into rows, at sizes where a block takes several runs, where runs are rounded to whole
lines, where few tiles are cut into slices, and where outputs are stored past the caches.  Smaller calls take a row
per lane: the two are compared over the whole range, and windows of it with the oracle."""
import numpy as np
import pytest

from paper_2412_04788_amd import guide, workloads as wl
from tests import bridge

pytestmark = pytest.mark.gpu
TOL = 1e-9
PAD = 256


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def _grid(nb, nm, rows):
    """A grid of at least `rows` rows with nb block sizes and nm token budgets."""
    rng = np.random.default_rng(nb * 100 + nm)
    blks = sorted(rng.choice(np.arange(1, 200), nb, replace=False).tolist())
    mbts = sorted(rng.choice(np.arange(100, 9000), nm, replace=False).tolist())
    per_hw = 5 * 11 * 8 * 8 * 3 * 2 * nb * nm
    hw = -(-rows // per_hw)
    assert hw <= 64
    return wl.make_grid(wl.MODELS_FULL, wl.hw_profiles(3, hw), wl.Axis.geom2(1, 11),
                        wl.Axis.table([17, 64, 129, 300, 640, 1111, 2000, 5000]),
                        wl.Axis.table([1, 2, 50, 99, 333, 500, 700, 1000]), wl.Axis.table([1, 3, 8]), wl.Axis.table([16, 4]),
                        wl.Axis.table(blks), wl.Axis.table(mbts))


def _padded(torch, names, n, dt):
    """Columns of n elements inside larger buffers that are filled with 7."""
    full = {k: torch.full((n + 2 * PAD,), 7, dtype=dt.get(k, torch.float64), device="cuda") for k in names}
    return full, {k: v[PAD:PAD + n] for k, v in full.items()}


def _untouched(full, n):
    return all(bool((v[:PAD] == 7).all()) and bool((v[PAD + n:] == 7).all()) for v in full.values())


def _windows(n, k, size=200):
    at = np.linspace(0, n - size, k).astype(np.int64)
    return sorted(set(at.tolist()))


METRIC_DT = {"b_max": "int32", "feasible": "uint8"}


# (tiles of a block above a run's most: 5 x 6 from 87 040 tiles on, 64 x 3 and 3 x 64 from 8192; 1 x 5: runs rounded down to
# a multiple of 64; 64 x 64: slices, and single tiles; 40 bytes a row are stored past the caches from 1.68 million rows on)
@pytest.mark.parametrize("nb,nm,n,first,tm", [(5, 6, 3_200_001, 777, 0), (5, 6, 2_700_000, 0, 1), (64, 3, 1_750_003, 193, 0),
                                              (3, 64, 1_620_000, 0, 1), (3, 64, 1_700_000, 64, 0), (64, 64, 200_017, 4097, 0),
                                              (64, 64, 140_000, 0, 1), (64, 64, 1_300_000, 999, 1), (5, 1, 300_001, 3, 0),
                                              (1, 5, 5_000_000, 1, 1), (8, 8, 131_073, 0, 0)])
def test_wide_grid(ora, torch_cuda, nb, nm, n, first, tm):
    torch = torch_cuda
    g = _grid(nb, nm, first + n)
    ctx, gg = bridge.gpu_context(g), bridge.gpu_grid(g)
    full, out = _padded(torch, guide.METRIC_COLUMNS, n, {k: getattr(torch, v) for k, v in METRIC_DT.items()})
    ctx.eval_grid(gg, first, n, out=out, time_model=tm)
    part_full, part = _padded(torch, guide.METRIC_COLUMNS, 131_072, {k: getattr(torch, v) for k, v in METRIC_DT.items()})
    for at in range(0, n, 131_072):
        m = min(131_072, n - at)
        ctx.eval_grid(gg, first + at, m, out={k: v[:m] for k, v in part.items()}, time_model=tm)
        for k in out:
            assert torch.equal(out[k][at:at + m], part[k][:m]), (k, at)
    assert _untouched(full, n)
    for at in _windows(n, 12):
        exp = ora.eval_grid(bridge.ora_grid(g), first + at, 200, time_model=tm)
        for k in out:
            got = bridge.to_np(out[k][at:at + 200].clone(), np.uint32 if k == "b_max" else None)
            if got.dtype == np.float64:
                assert bridge.rel_err(got, exp[k]).max() <= TOL, k
            else:
                np.testing.assert_array_equal(got, exp[k])


def test_wide_grid_without_some_columns(torch_cuda):
    torch = torch_cuda
    n, g = 300_000, _grid(5, 6, 300_100)
    ctx, gg = bridge.gpu_context(g), bridge.gpu_grid(g)
    dt = {k: getattr(torch, v) for k, v in METRIC_DT.items()}
    _, whole = _padded(torch, guide.METRIC_COLUMNS, n, dt)
    ctx.eval_grid(gg, 100, n, out=whole)
    for names in (("feasible",), ("t_batch", "b_max"), ("cost",)):
        full, out = _padded(torch, names, n, dt)
        ctx.eval_grid(gg, 100, n, out=out)
        assert all(torch.equal(out[k], whole[k]) for k in names) and _untouched(full, n)


def test_few_wide_tiles_use_the_chip(torch_cuda):
    """A call over 49 tiles of 64 x 64 rows costs about what the same number of rows in tiles of 8 x 8 costs (1.6 times with
    a block per tile)."""
    torch, times, n = torch_cuda, [], 200_000
    for nb, nm in ((64, 64), (8, 8)):
        g = _grid(nb, nm, n)
        ctx, out = bridge.gpu_context(g), bridge.metric_buffers(n)
        call, t = ctx.prepared("eval_grid", bridge.gpu_grid(g), 0, n, out=out), []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(200):
                call()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        times.append(min(t))
    assert times[0] <= 1.35 * times[1], times


EXTRAS_DT = {"max_parallelism": "int64", "cluster_tok_s": "float64", "paper_tok_s": "float64", "feasible_kept": "uint8"}


# (56 bytes a row are stored past the caches from 1.2 million rows on where runs start on whole lines; 249 999 and 250 000
# rows lie on either side of the rule for all columns, 699 999 and 700 000 for one narrow column of 3 x 4 tiles)
@pytest.mark.parametrize("nb,nm,n,first,tm,names", [
    (2, 3, 1_250_001, 0, 0, None), (2, 3, 1_900_000, 777, 1, None), (5, 6, 250_000, 41, 0, None), (5, 6, 249_999, 41, 0, None),
    (5, 6, 3_000_000, 30, 1, None), (64, 3, 1_700_011, 192, 0, None), (1, 64, 700_003, 5, 0, None), (64, 64, 260_001, 4097, 1, None),
    (64, 64, 1_300_000, 0, 0, None), (2, 2, 420_000, 1, 0, ("cluster_tok_s", "feasible_kept")), (6, 1, 450_000, 0, 0, None),
    (3, 4, 700_000, 13, 0, ("s_adj",)), (3, 4, 699_999, 13, 0, ("s_adj",)), (4, 4, 500_001, 0, 0, ("n_segments", "b_max_kept")),
    (2, 3, 1_800_005, 6, 0, ("max_parallelism",)), (1, 2, 500_000, 1, 0, None)])
def test_cluster_columns(ora, torch_cuda, nb, nm, n, first, tm, names):
    torch = torch_cuda
    names, g, keep = names or guide.EXTRAS_COLUMNS, _grid(nb, nm, first + n), 0.3
    dt = {k: getattr(torch, EXTRAS_DT.get(k, "int32")) for k in guide.EXTRAS_COLUMNS}
    ctx, gg = bridge.gpu_context(g), bridge.gpu_grid(g)
    full, out = _padded(torch, names, n, dt)
    ctx.eval_extras(gg, first, n, 13, out, time_model=tm, kv_keep=keep)
    step = 200_000                                              # a row per lane, whatever the columns
    _, part = _padded(torch, guide.EXTRAS_COLUMNS, step, dt)
    for at in range(0, n, step):
        m = min(step, n - at)
        ctx.eval_extras(gg, first + at, m, 13, {k: v[:m] for k, v in part.items()}, time_model=tm, kv_keep=keep)
        for k in out:
            assert torch.equal(out[k][at:at + m], part[k][:m]), (k, at)
    assert _untouched(full, n)
    for at in _windows(n, 12):
        exp = ora.eval_extras_grid(bridge.ora_grid(g), 13, first + at, 200, time_model=tm, kv_keep=keep)
        for k in out:
            got = out[k][at:at + 200].cpu().numpy()
            if got.dtype == np.float64:
                assert bridge.rel_err(got, exp[k]).max() <= TOL, k
            else:
                np.testing.assert_array_equal(got.astype(np.int64) & (0xFFFFFFFF if got.dtype == np.int32 else -1),
                                              np.asarray(exp[k]).astype(np.int64), err_msg=k)


def test_ragged_ranges_cost_about_as_much_as_whole_ones(torch_cuda):
    """Blocks whose runs share lines at their ends store through the caches (stores past them: 1.55 times the time)."""
    torch, times, n = torch_cuda, [], 1_900_000
    dt = {k: getattr(torch, EXTRAS_DT.get(k, "int32")) for k in guide.EXTRAS_COLUMNS}
    g = _grid(2, 3, n + 777)
    ctx, out = bridge.gpu_context(g), {k: torch.zeros(n, dtype=dt[k], device="cuda") for k in guide.EXTRAS_COLUMNS}
    for first in (0, 777):
        call, t = ctx.prepared("eval_extras", bridge.gpu_grid(g), first, n, 8, out), []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(50):
                call()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        times.append(min(t))
    assert times[1] <= 1.25 * times[0], times
