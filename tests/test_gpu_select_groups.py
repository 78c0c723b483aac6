"""Grouped top-k (one pass with per-wave lists) at the edges of its batches, for every list width and with the row orders
that are worst for it, against the oracle's linear scan.  Values are copied and rows compared, so everything is exact."""
import numpy as np
import pytest

from paper_2412_04788_amd import guide
from tests.test_gpu_select import _topk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    from paper_2412_04788_amd import workloads as wl
    assert torch.cuda.is_available()
    ctx = guide.Context(0)
    ctx.set_models(wl.models_array([wl.DENSE_7B]))
    ctx.set_hardware(wl.hw_array([wl.HW_TINY]))
    return torch, ctx


def _check(ora, setup, obj, grp, G, k, feasible=None, cons=()):
    torch, ctx = setup
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()        # noqa: E731
    i, v, c = _topk(torch, ctx, dev(obj), k=k, feasible=None if feasible is None else dev(feasible),
                    constraints=[(dev(col), cap) for col, cap in cons], group=dev(grp.astype(np.int32)), n_groups=G)
    ei, ev, ec = ora.select_topk(obj, feasible, list(cons), group=grp.astype(np.uint32), n_groups=G, k=k)
    np.testing.assert_array_equal(c, ec)
    np.testing.assert_array_equal(i, ei)
    np.testing.assert_array_equal(v, ev)


@pytest.mark.parametrize("n", [1, 7, 4095, 4096, 4097, 40_000, 600_001])
@pytest.mark.parametrize("G,k", [(1, 1), (64, 1), (3, 2), (10, 3), (64, 4), (64, 8), (5, 7)])
def test_batch_edges_and_list_widths(ora, setup, n, G, k):
    rng = np.random.default_rng(n * 100 + G + k)
    obj = np.repeat(np.round(rng.standard_normal(n // 4 + 1), 3), 4)[:n]            # runs of equal values, many ties
    grp = rng.integers(0, G + (2 if G > 1 else 0), n)                               # ids from G on are ignored
    fe = (rng.random(n) < 0.7).astype(np.uint8)
    cons = [(rng.random(n), 0.8), (rng.random(n), 0.9), (rng.random(n), 0.95)][:k % 4]
    _check(ora, setup, obj, grp, G, k, fe, cons)


@pytest.mark.parametrize("order", ["ascending", "descending", "equal", "special"])
def test_row_orders(ora, setup, order):
    n, G = 50_000, 6
    rng = np.random.default_rng(3)
    obj = {"ascending": np.arange(n) * 1.0, "descending": -np.arange(n) * 1.0, "equal": np.zeros(n),
           "special": rng.choice([np.inf, -np.inf, np.nan, 0.0, -0.0, 5e-324, -1.0], n)}[order]
    grp = np.arange(n) * G // n if order == "equal" else rng.integers(0, G, n)
    for k in (1, 3, 8):
        _check(ora, setup, obj, grp, G, k)


def test_groups_without_passing_rows(ora, setup):
    n = 5000
    _check(ora, setup, np.arange(n) * 1.0, np.full(n, 2), 4, 3)
    _check(ora, setup, np.arange(n) * 1.0, np.full(n, 2), 4, 3, np.zeros(n, dtype=np.uint8))
    _check(ora, setup, np.full(n, np.nan), np.zeros(n, dtype=np.int64), 2, 2)


@pytest.mark.parametrize("k", [1, 3, 8])
@pytest.mark.parametrize("order", ["falling", "equal"])
def test_no_row_order_is_much_slower_than_another(setup, order, k):
    """Columns that fall with the row number and columns of equal values cost about what random ones do (a list that every
    row enters one after the other made them up to eighteen times as slow)."""
    torch, ctx = setup
    n, G = 4_000_000, 5
    grp = torch.randint(0, G, (n,), dtype=torch.int32, device="cuda")
    cols = {"random": torch.rand(n, dtype=torch.float64, device="cuda"), "equal": torch.zeros(n, dtype=torch.float64, device="cuda"),
            "falling": -torch.arange(n, dtype=torch.float64, device="cuda")}
    idx = torch.zeros(G * k, dtype=torch.int64, device="cuda")
    val, cnt = torch.zeros(G * k, dtype=torch.float64, device="cuda"), torch.zeros(G, dtype=torch.int64, device="cuda")
    ws = torch.empty(ctx.select_workspace_bytes(guide.SELECT_TOPK, n, G), dtype=torch.uint8, device="cuda")

    def best(col):
        call, t = ctx.prepared("select", guide.SELECT_TOPK, n, cols[col], idx, val, cnt, ws, group=grp, n_groups=G, k=k), []
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                call()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)
    random, other = best("random"), best(order)
    assert other <= 3.0 * random, (other, random)
