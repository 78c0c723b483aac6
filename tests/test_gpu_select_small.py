"""Selections over at most 4096 rows take one launch without sample and filter pass: the edges of that path, next to the
general one just above it, against the oracle."""
import numpy as np
import pytest

from paper_2412_04788_amd import guide, workloads as wl
from tests import bridge
from tests.test_gpu_select import _pareto, _topk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    assert torch.cuda.is_available()
    ctx = guide.Context(0)
    return torch, ctx


def _data(kind, n, rng):
    if kind == "cloud":
        return rng.random(n), rng.random(n)
    if kind == "front":                                 # every row is on it
        x = rng.permutation(n) * 1.0
        return x, -x
    if kind == "ties":
        return np.round(rng.random(n), 1), np.round(rng.random(n), 1)
    if kind == "one x":
        return np.full(n, 3.0), np.round(rng.random(n), 2)
    return rng.choice([np.inf, -np.inf, np.nan, 0.0, -0.0, 1.0, 5e-324], n), rng.choice([np.inf, -1.0, 0.0, np.nan, 2.0], n)


@pytest.mark.parametrize("n", [1, 2, 63, 1000, 1025, 4095, 4096, 4097])
@pytest.mark.parametrize("kind", ["cloud", "front", "ties", "one x", "special"])
def test_small_pareto_and_topk(ora, setup, n, kind):
    torch, ctx = setup
    rng = np.random.default_rng(n)
    x, y = _data(kind, n, rng)
    c = rng.random(n)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()        # noqa: E731
    dx, dy, dc = dev(x), dev(y), dev(c)
    for fe, cons in ((None, []), ((rng.random(n) < 0.6).astype(np.uint8), [(c, 0.7)]), (np.zeros(n, np.uint8), [])):
        dcons = [(dc, cap) for _, cap in cons]
        dfe = None if fe is None else dev(fe)
        mask = (np.ones(n, bool) if fe is None else fe != 0) & ~np.isnan(x) & ~np.isnan(y)
        for col, cap in cons:
            mask &= col <= cap
        exp = ora.pareto_brute(x, y, mask.astype(np.uint8))
        got, m = _pareto(torch, ctx, dx, dy, dfe, dcons)
        assert m == len(exp)
        np.testing.assert_array_equal(got, exp)
        got, m = _pareto(torch, ctx, dx, dy, dfe, dcons, capacity=3)
        assert m == len(exp)
        np.testing.assert_array_equal(got, exp[:3])
        for k in (1, 2, 3, 4, 5):
            i, v, cnt = _topk(torch, ctx, dx, k=k, feasible=dfe, constraints=dcons)
            ei, ev, ec = ora.select_topk(x, fe, cons, k=k)
            np.testing.assert_array_equal(i, ei)
            np.testing.assert_array_equal(v, ev)
            np.testing.assert_array_equal(cnt, ec)


@pytest.mark.parametrize("k", [1, 4, 8])
@pytest.mark.parametrize("count", [1, 1080, 4096, 4100])
def test_small_evaluate_and_select_equals_the_separate_calls(setup, k, count):
    torch, _ = setup
    g = wl.grid_full()
    ctx = bridge.gpu_context(g)
    gg, first = bridge.gpu_grid(g), 700_001
    out = bridge.metric_buffers(count)
    z = lambda n, dt: torch.full((n,), -7, dtype=dt, device="cuda")         # noqa: E731
    res = [(z(k, torch.int64), z(k, torch.float64), z(1, torch.int64), z(count, torch.int64), z(1, torch.int64)) for _ in range(2)]
    ti, tv, tc, pi, pc = res[0]
    sels = [ctx.column_select(guide.SELECT_TOPK, "cost", ti, tv, tc, constraints=[("t_prefill", 5.0)], k=k),
            ctx.column_select(guide.SELECT_PARETO, "t_prefill", pi, None, pc, objective_y="cost", capacity=count)]
    ws = torch.empty(ctx.eval_select_workspace_bytes(sels, count), dtype=torch.uint8, device="cuda")
    ctx.eval_select(gg, first, count, out, sels, ws)
    ti, tv, tc, pi, pc = res[1]
    ctx.select(guide.SELECT_TOPK, count, out["cost"], ti, tv, tc, ws, feasible=out["feasible"],
               constraints=[(out["t_prefill"], 5.0)], k=k)
    ctx.select(guide.SELECT_PARETO, count, out["t_prefill"], pi, None, pc, ws, objective_y=out["cost"],
               feasible=out["feasible"], capacity=count)
    torch.cuda.synchronize()
    for a, b in zip(*res):
        assert torch.equal(a, b)
