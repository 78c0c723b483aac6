"""Grids with many values on the two fastest axes, and the cluster-level columns, at sizes that take a row per lane: ragged
ranges, tables beyond LDS and missing columns, against the oracle."""
import numpy as np
import pytest

from paper_2412_04788_amd import guide, workloads as wl
from tests import bridge

pytestmark = pytest.mark.gpu
TOL = 1e-9
FLOATS = ("t_prefill", "t_decode", "t_batch", "decode_tok_s", "cost")


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def _grid(nb, nm, slow=1):
    rng = np.random.default_rng(nb * 100 + nm)
    blks = sorted(rng.choice(np.arange(1, 200), nb, replace=False).tolist())
    mbts = sorted(rng.choice(np.arange(100, 9000), nm, replace=False).tolist())
    return wl.make_grid([wl.DENSE_7B, wl.MOE_8X], wl.hw_profiles(3, 2), wl.Axis.table([1, 5, 37, 300][:1 + slow]),
                        wl.Axis.table([17, 640, 5000]), wl.Axis.table([1, 2, 333]), wl.Axis.table([1, 3]),
                        wl.Axis.table([16, 4]), wl.Axis.table(blks), wl.Axis.table(mbts))


def _check_metrics(torch, ora, g, first, count, tm, names=None):
    n = count
    out = bridge.metric_buffers(n)
    for v in out.values():
        v.fill_(7)
    used = {k: v for k, v in out.items() if names is None or k in names}
    bridge.gpu_context(g).eval_grid(bridge.gpu_grid(g), first, n, out=used, time_model=tm)
    torch.cuda.synchronize()
    exp = ora.eval_grid(bridge.ora_grid(g), first, n, time_model=tm)
    for k in out:
        got = bridge.to_np(out[k], np.uint32 if k == "b_max" else None)
        if k not in used:
            assert (got == 7).all(), k
        elif k in FLOATS:
            assert bridge.rel_err(got, exp[k]).max() <= TOL, k
        else:
            np.testing.assert_array_equal(got, exp[k])


@pytest.mark.parametrize("nb,nm", [(5, 1), (1, 5), (5, 6), (2, 7), (64, 3), (3, 64), (64, 64)])
@pytest.mark.parametrize("tm", [0, 1])
def test_wide_axes(ora, torch_cuda, nb, nm, tm):
    g = _grid(nb, nm, 0 if nb * nm > 1000 else 3)
    size = min(g.size, 60_000)
    _check_metrics(torch_cuda, ora, g, 0, size, tm)
    first = nb * nm + 1 if nb * nm > 1 else 1
    for count in (1, nb * nm - 1, nb * nm, 3 * nb * nm + 5, min(g.size - first, 20_003)):
        _check_metrics(torch_cuda, ora, g, first, count, tm)
    _check_metrics(torch_cuda, ora, g, 2, 501, tm, names=("t_batch", "feasible"))


def test_wide_axes_with_more_coefficient_rows_than_lds(ora, torch_cuda):
    models = [wl.DENSE_7B, wl.DENSE_13B, wl.DENSE_34B, wl.DENSE_70B, wl.MOE_8X]
    g = wl.make_grid(models, wl.hw_profiles(9, 1), wl.Axis.table([3]), wl.Axis.table([100, 7000]), wl.Axis.table([50]),
                     wl.Axis.table([1, 2, 3, 4, 5, 6, 8]), wl.Axis.table([16, 8, 4]), wl.Axis.table([1, 7, 16, 24, 32]),
                     wl.Axis.table([500, 2048, 8192]))
    assert 5 * 7 * 3 > 96
    _check_metrics(torch_cuda, ora, g, 0, g.size, 0)
    _check_metrics(torch_cuda, ora, g, 11, g.size - 29, 1)


@pytest.mark.parametrize("nb,nm", [(1, 1), (2, 3), (5, 6), (64, 2), (64, 64)])
@pytest.mark.parametrize("ragged", [False, True])
def test_cluster_columns(ora, torch_cuda, nb, nm, ragged):
    torch = torch_cuda
    g = _grid(nb, nm, 0 if nb * nm > 1000 else 3)
    first = 1 + nb * nm // 2 if ragged else 0
    n = min(g.size - first, 50_000) - (3 if ragged else 0)
    dt = {"max_parallelism": torch.int64, "cluster_tok_s": torch.float64, "paper_tok_s": torch.float64,
          "feasible_kept": torch.uint8}
    for tm, keep in ((0, 0.0), (1, 0.3)):
        out = {k: torch.full((n,), 9, dtype=dt.get(k, torch.int32), device="cuda") for k in guide.EXTRAS_COLUMNS}
        bridge.gpu_context(g).eval_extras(bridge.gpu_grid(g), first, n, 13, out, time_model=tm, kv_keep=keep)
        torch.cuda.synchronize()
        exp = ora.eval_extras_grid(bridge.ora_grid(g), 13, first, n, time_model=tm, kv_keep=keep if keep else 1.0)
        for k in guide.EXTRAS_COLUMNS:
            got = out[k].cpu().numpy()
            if got.dtype == np.float64:
                assert bridge.rel_err(got, exp[k]).max() <= TOL, k
            else:
                np.testing.assert_array_equal(got.astype(np.int64) & (0xFFFFFFFF if got.dtype == np.int32 else -1),
                                              np.asarray(exp[k]).astype(np.int64), err_msg=k)
