"""guide_simulate by the queue that holds the decoders: slots in LDS (one, two and three levels of minima), slots whose lane
runs far more sequences than it expects (the rest in global memory), heaps where the lanes of a block expect more than LDS holds; and
at the ends of the launch shapes.  Against the CPU oracle's step-level simulator."""
import numpy as np
import pytest

from paper_2412_04788_amd import guide, workloads as wl
from tests import bridge
from tests.test_gpu_simulate import _compare, _run
from tests.test_gpu_simulate_paths import CLOSED, _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def _grid(batch):
    hw = wl.Hardware(2e15, 8e12, 4000 * wl.GIB, 6e11)
    return wl.make_grid([wl.DENSE_7B, wl.MOE_8X], [hw], wl.Axis.table(batch), wl.Axis.table([1]), wl.Axis.table([1]),
                        wl.Axis.table([1, 2]), wl.Axis.table([16, 8]), wl.Axis.table([16]), wl.Axis.table([8192, 2048]))


# the most decoders: one block of slots and one more, four blocks, sixteen, and all of three levels
@pytest.mark.parametrize("cap", [1, 16, 17, 64, 65, 256, 257, 1024])
def test_levels_of_the_slots(ora, torch_cuda, cap):
    rng = np.random.default_rng(cap)
    n = 1024
    tr = wl.Trace(np.sort(rng.random(n) * 2.0), rng.integers(8, 64, n).astype(np.uint32), rng.integers(1, 500, n).astype(np.uint32))
    g = _grid([cap, max(cap - 3, 1)])
    idx = np.arange(g.size, dtype=np.uint32)
    _check(torch_cuda, ora, g, idx, np.where(idx % 2 == 0, 1e6, 30.0), tr)


# (lists of one lane per wave hold every decoder in their slots; in longer ones, 300 requests at the start of a trace that ends
# a long time after make lanes expect one sequence and run 300)
@pytest.mark.parametrize("n_cfg", [40, 2500])
def test_more_decoders_than_expected(ora, torch_cuda, n_cfg):
    rng = np.random.default_rng(n_cfg)
    n = 320
    t = np.concatenate([np.sort(rng.random(300)), 1e7 + np.arange(20.0)])
    tr = wl.Trace(t, rng.integers(8, 300, n).astype(np.uint32), rng.integers(1, 700, n).astype(np.uint32))
    g = _grid([1024, 33, 200, 7])
    idx = (np.arange(n_cfg) % g.size).astype(np.uint32)
    rate = 1.0 + (np.arange(n_cfg) % 97) * 3.0
    pick = np.unique(np.linspace(0, n_cfg - 1, 40).astype(np.int64))
    _check(torch_cuda, ora, g, idx, rate, tr, pick)


@pytest.mark.parametrize("n_cfg", [256, 640, 641, 2048, 2049, 16384, 16385, 49153])
def test_launch_shapes(ora, torch_cuda, n_cfg):
    g = wl.grid_full()
    tr = wl.request_trace(n=40, seed=n_cfg)
    idx, rate = wl.sim_configs(g, n_cfg, seed=n_cfg)
    pick = np.unique(np.concatenate([np.linspace(0, n_cfg - 1, 64), [n_cfg - 2, n_cfg - 1]]).astype(np.int64))
    _check(torch_cuda, ora, g, idx, rate, tr, pick)
    # a configuration's results are the same bits in every list
    ctx = bridge.gpu_context(g)
    whole, part = (_run(torch_cuda, ctx, g, idx[p], rate[p], tr) for p in (np.arange(n_cfg), pick))
    for k in whole:
        np.testing.assert_array_equal(whole[k][pick], part[k])


# lists are ordered from 64 requests on where blocks have several waves, and where LDS has no slot for every request in blocks of one
@pytest.mark.parametrize("n_cfg, n_req", [(16385, 63), (16385, 64), (2049, 352), (2049, 353)])
def test_the_line_of_ordering(ora, torch_cuda, n_cfg, n_req):
    g = wl.grid_full()
    tr = wl.request_trace(n=n_req, seed=n_cfg)
    idx, rate = wl.sim_configs(g, n_cfg, seed=n_req)
    pick = np.unique(np.linspace(0, n_cfg - 1, 48).astype(np.int64))
    _check(torch_cuda, ora, g, idx, rate, tr, pick)


# values per lane of the percentiles' sorting network: 1, 2, 4, 8, 16
@pytest.mark.parametrize("n_req", [2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1000])
def test_percentiles_by_trace_length(ora, torch_cuda, n_req):
    g = wl.grid_full()
    tr = wl.request_trace(n=n_req, seed=n_req)
    idx, rate = wl.sim_configs(g, 70, seed=n_req)
    _check(torch_cuda, ora, g, idx, rate, tr, np.arange(0, 70, 3))


@pytest.mark.parametrize("n_req", [7, 100, 400, 1000])
def test_percentiles_of_infinite_waits(torch_cuda, n_req):
    """Arrivals over rate that are infinite: those requests' times to the first token (infinity less infinity) count as infinite."""
    hw = wl.Hardware(1e15, 5e12, 1e6 * wl.GIB, 4e11)
    g = wl.make_grid([wl.DENSE_7B], [hw], wl.Axis.table([1, 2]), wl.Axis.table([1]), wl.Axis.table([1]),
                     wl.Axis.table([1, 4]), wl.Axis.table([16]), wl.Axis.table([16]), wl.Axis.table([512, 8192]))
    rng = np.random.default_rng(n_req)
    finite = (n_req + 1) // 2                           # the median is the greatest of theirs
    t = np.concatenate([np.arange(finite) * 1e-10, np.full(n_req - finite, 1e300)])
    n_in, n_out = rng.integers(5, 900, n_req).astype(np.uint32), rng.integers(1, 400, n_req).astype(np.uint32)
    idx, rate = np.arange(g.size, dtype=np.uint32), np.full(g.size, 1e-10)
    ctx = bridge.gpu_context(g)
    for sched in (0, 1):
        got = _run(torch_cuda, ctx, g, idx, rate, wl.Trace(t, n_in, n_out), scheduler=sched)
        few = _run(torch_cuda, ctx, g, idx, rate, wl.Trace(t[:finite], n_in[:finite], n_out[:finite]), scheduler=sched)
        assert np.all(got["status"] == 0) and np.all(got["ttft_p99"] == np.inf)
        assert np.all(np.isfinite(got["ttft_p50"])) and np.all(got["ttft_p50"] >= few["ttft_p99"])
        if finite < 100:                                # (the 99th percentile is the greatest)
            np.testing.assert_array_equal(got["ttft_p50"], few["ttft_p99"])


# (32-bit and 64-bit keys)
@pytest.mark.parametrize("n_out", [1_000_000, 1 << 24])
def test_arrivals_beyond_the_range_of_doubles(ora, torch_cuda, n_out):
    """Arrivals over rate that are infinite: the clock is infinite from there on, and every request still runs.  A run of decode
    steps while others wait for a place is advanced at once (step by step it would take seconds here, a minute with 64-bit keys)."""
    hw = wl.Hardware(1e15, 5e12, 1e6 * wl.GIB, 4e11)
    g = wl.make_grid([wl.DENSE_7B], [hw], wl.Axis.table([1, 2]), wl.Axis.table([1]), wl.Axis.table([1]),
                     wl.Axis.table([1, 4]), wl.Axis.table([16]), wl.Axis.table([16]), wl.Axis.table([512, 8192]))
    idx = np.arange(g.size, dtype=np.uint32)
    rate = np.full(g.size, 1e-10)
    t = np.array([0.0, 1e-10, 2e-10, 3e-10, 1e300, 1e300, 1.5e300])
    n_in, outs = np.array([700, 30, 5, 900, 8, 9, 10], dtype=np.uint32), np.array([3, 40, 1, 7, n_out, n_out, n_out], dtype=np.uint32)
    ctx, og = bridge.gpu_context(g), bridge.ora_grid(g)
    for sched in (0, 1):
        _run(torch_cuda, ctx, g, idx, rate, wl.Trace(t[:4], n_in[:4], outs[:4]), scheduler=sched)          # (loads the kernel)
        e = [torch_cuda.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        got = _run(torch_cuda, ctx, g, idx, rate, wl.Trace(t, n_in, outs), scheduler=sched)
        e[1].record()
        torch_cuda.cuda.synchronize()
        assert e[0].elapsed_time(e[1]) < 1000.0
        exp = ora.simulate_grid(og, idx, rate, t, n_in, outs, scheduler=sched | CLOSED)
        few = _run(torch_cuda, ctx, g, idx, rate, wl.Trace(t[:4], n_in[:4], outs[:4]), scheduler=sched)
        for k in ("status", "n_steps", "n_request_steps"):
            np.testing.assert_array_equal(got[k], exp[k], err_msg=k)
        assert np.all(got["status"] == 0) and np.all(got["tokens_s"] == 0.0)
        # four of the seven waited for finite times; the others count as infinite
        np.testing.assert_array_equal(got["ttft_p50"], few["ttft_p99"])
        assert np.all(np.isfinite(few["ttft_p99"])) and np.all(got["ttft_p99"] == np.inf)


# (also the additive model, whole prompts first, and generations that take 64-bit keys)
@pytest.mark.parametrize("n_cfg,n_req,tm,sched,longer", [(50_000, 127, 0, 0, 1), (50_000, 128, 0, 0, 1), (49_153, 129, 0, 0, 1), (70_001, 64, 0, 0, 1),
                                                         (20_000, 512, 0, 0, 1), (20_000, 513, 0, 0, 1), (33_000, 600, 0, 0, 1),
                                                         (66_000, 159, 0, 0, 1), (66_000, 160, 0, 0, 1), (49_153, 287, 0, 0, 1), (49_153, 288, 0, 0, 1),
                                                         (65_537, 257, 0, 0, 1), (49_999, 170, 1, 0, 1), (49_999, 170, 1, 1, 1), (49_999, 170, 0, 1, 1),
                                                         (49_157, 190, 0, 0, 300), (49_157, 190, 0, 1, 300), (49_157, 190, 1, 0, 300),
                                                         (256, 64, 0, 0, 1), (256, 65, 0, 0, 1), (257, 65, 0, 0, 1)])
def test_percentiles_by_the_waves_and_by_their_own_kernel(ora, torch_cuda, n_cfg, n_req, tm, sched, longer):
    """Percentiles come from the simulation's waves, but for those of the longest configurations or of short traces: the same bits as
    in a list of one lane per wave, whose waves work out all of them."""
    torch = torch_cuda
    tr = wl.request_trace(n=n_req, seed=n_req)
    if longer == 1:
        g = wl.grid_full()
        idx, rate = wl.sim_configs(g, n_cfg, seed=n_req)
    else:                                               # (a pool that holds them)
        tr = wl.Trace(tr.arrival_unit, tr.n_in, tr.n_out * np.uint32(longer))
        g = _grid([1, 9, 60, 700])
        idx = (np.arange(n_cfg) * 7 % g.size).astype(np.uint32)
        rate = 1e-4 * 1.001 ** (np.arange(n_cfg) % 5000)
        assert int(tr.n_out.sum()) > 1 << 22
    ctx = bridge.gpu_context(g)
    whole = _run(torch, ctx, g, idx, rate, tr, time_model=tm, scheduler=sched)
    assert (whole["status"] == guide.SIM_OK).sum() > n_cfg // 2
    pick = np.unique(np.linspace(0, n_cfg - 1, 1500).astype(np.int64))
    part = _run(torch, ctx, g, np.ascontiguousarray(idx[pick]), np.ascontiguousarray(rate[pick]), tr, time_model=tm, scheduler=sched)
    for k in whole:
        np.testing.assert_array_equal(whole[k][pick], part[k], err_msg=k)
    # every configuration that ended has its percentiles, whichever kernel wrote them
    ok = whole["status"] == guide.SIM_OK
    assert np.all(np.isfinite(whole["ttft_p99"][ok])) and np.all(whole["ttft_p50"][ok] <= whole["ttft_p99"][ok])
    assert np.all(np.isinf(whole["ttft_p50"][~ok]))
    if longer == 1:                                     # (a clock of 10^6 s has no 1e-9 of a TTFT of milliseconds)
        few = pick[::125]
        exp = ora.simulate_grid(bridge.ora_grid(g), idx[few], rate[few], tr.arrival_unit, tr.n_in, tr.n_out, time_model=tm, scheduler=sched)
        _compare({k: v[few] for k, v in whole.items()}, exp)
