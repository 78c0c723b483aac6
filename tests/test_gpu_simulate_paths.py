"""guide_simulate where its kernel takes another path: wave occupancy by the number of configurations, heaps that spill
out of LDS, 64-bit keys and counters, step times that are not linear in the context, arrival rates at the ends of the
range.  All against the CPU oracle's step-level simulator."""
import numpy as np
import pytest

from paper_2412_04788_amd import guide, workloads as wl
from tests import bridge
from tests.test_gpu_simulate import _compare, _run

pytestmark = pytest.mark.gpu
CLOSED = guide.SIM_CLOSED_FORM_RUNS


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def _check(torch, ora, g, idx, rate, tr, pick=None, scheds=(0, 1), time_model=0):
    ctx, og = bridge.gpu_context(g), bridge.ora_grid(g)
    pick = np.arange(len(idx)) if pick is None else pick
    for sched in scheds:
        got = _run(torch, ctx, g, idx, rate, tr, time_model=time_model, scheduler=sched)
        # the closed-form option is accepted and changes nothing
        flagged = _run(torch, ctx, g, idx, rate, tr, time_model=time_model, scheduler=sched | CLOSED)
        for k in got:
            np.testing.assert_array_equal(flagged[k], got[k], err_msg=k)
        exp = ora.simulate_grid(og, idx[pick], rate[pick], tr.arrival_unit, tr.n_in, tr.n_out, scheduler=sched & 1,
                                time_model=time_model)
        _compare({k: v[pick] for k, v in got.items()}, exp)


@pytest.mark.parametrize("n_req", [1, 15, 16, 23])
@pytest.mark.parametrize("n_cfg", [1, 63, 1024, 1025, 2048, 2049, 33000])
def test_lanes_per_wave_by_configuration_count(ora, torch_cuda, n_cfg, n_req):
    g = wl.grid_full()
    tr = wl.request_trace(n=n_req, seed=n_cfg)
    idx, rate = wl.sim_configs(g, n_cfg, seed=n_cfg)
    pick = np.unique(np.linspace(0, n_cfg - 1, min(n_cfg, 96)).astype(np.int64))
    _check(torch_cuda, ora, g, idx, rate, tr, pick)


def test_heaps_that_do_not_fit_lds(ora, torch_cuda):
    """Every lane of the chip runs up to 1024 sequences at once, four to eight times what its LDS share holds."""
    hw = wl.Hardware(2e15, 8e12, 4000 * wl.GIB, 6e11)
    g = wl.make_grid([wl.DENSE_7B, wl.MOE_8X], [hw], wl.Axis.table([1024, 700]), wl.Axis.table([1]), wl.Axis.table([1]),
                     wl.Axis.table([1, 2]), wl.Axis.table([16, 8]), wl.Axis.table([16]), wl.Axis.table([8192, 2048]))
    rng = np.random.default_rng(5)
    n = 1024
    tr = wl.Trace(np.sort(rng.random(n) * 3.0), rng.integers(8, 64, n).astype(np.uint32), rng.integers(1, 400, n).astype(np.uint32))
    n_cfg = 65536
    idx = (np.arange(n_cfg) % g.size).astype(np.uint32)
    rate = np.where(np.arange(n_cfg) % 3 == 0, 64.0, 1e6 + np.arange(n_cfg))
    _check(torch_cuda, ora, g, idx, rate, tr, np.linspace(0, n_cfg - 1, 24).astype(np.int64))


def test_long_generations_take_64_bit_keys(ora, torch_cuda):
    hw = wl.Hardware(1e15, 5e12, 1e6 * wl.GIB, 4e11)
    g = wl.make_grid([wl.DENSE_7B], [hw], wl.Axis.table([1, 3, 64]), wl.Axis.table([1]), wl.Axis.table([1]),
                     wl.Axis.table([1, 4]), wl.Axis.table([16]), wl.Axis.table([16]), wl.Axis.table([512, 8192]))
    n_out = np.array([1 << 20, 1 << 20, 700_001, 1, 1 << 20, 5, 400_000, 1 << 19], dtype=np.uint32)
    assert n_out.sum() >= 2 ** 22
    tr = wl.Trace(np.arange(8) * 0.25, np.array([7, 100, 9000, 3, 16, 1, 60_000, 250], dtype=np.uint32), n_out)
    idx = np.arange(g.size, dtype=np.uint32)
    # Arrivals within the first four seconds: TTFT = first token - arrival, and after n steps the two clocks may differ by
    # n 2^-53 of the clock (1e6 steps to 5000 s: 5e-7 s), which the 1e-9 allows for a TTFT of hours behind such
    # runs but not for one of milliseconds (an arrival at 1750 s read 2.9e-9 apart).
    _check(torch_cuda, ora, g, idx, np.where(idx % 2, 1.0, 0.5), tr)


def test_long_prompts_take_64_bit_counters(ora, torch_cuda):
    hw = wl.Hardware(1e15, 5e12, 1e9 * wl.GIB, 4e11)
    g = wl.make_grid([wl.DENSE_7B], [hw], wl.Axis.table([2, 40]), wl.Axis.table([1]), wl.Axis.table([1]),
                     wl.Axis.table([1]), wl.Axis.table([16]), wl.Axis.table([16]), wl.Axis.table([1 << 20, (1 << 32) - 1]))
    n = 72
    tr = wl.Trace(np.arange(n) * 1.0, np.full(n, 1 << 24, dtype=np.uint32), np.arange(1, n + 1, dtype=np.uint32))
    assert int(tr.n_in.astype(np.int64).sum()) >= 2 ** 30
    idx = np.arange(g.size, dtype=np.uint32)
    _check(torch_cuda, ora, g, idx, np.full(g.size, 0.01), tr)


def test_attention_bound_by_arithmetic(ora, torch_cuda):
    """Peak so low that attention turns from read bound to compute bound inside the runs: step times are not linear."""
    hws = [wl.Hardware(2e13, 4e12, 900 * wl.GIB, 4e11), wl.Hardware(1e13, 8e12, 900 * wl.GIB, 4e11), wl.HW_TINY]
    g = wl.make_grid([wl.DENSE_70B, wl.DENSE_7B], hws, wl.Axis.table([1, 5, 33]), wl.Axis.table([1]), wl.Axis.table([1]),
                     wl.Axis.table([1, 8]), wl.Axis.table([16, 4]), wl.Axis.table([16]), wl.Axis.table([2048]))
    tr = wl.request_trace(n=60, seed=3)
    idx = np.arange(g.size, dtype=np.uint32)
    rate = np.where(idx % 2, 0.05, 4.0)
    _check(torch_cuda, ora, g, idx, rate, tr)
    _check(torch_cuda, ora, g, idx, rate, tr, time_model=1)


def test_attention_that_turns_inside_a_run(ora, torch_cuda):
    """Attention turns from read bound to bound by arithmetic where context = r / (1 - r g), r = peak / bandwidth and g the
    share of the heads that are KV heads: 99 to 10 000 tokens here, in the middle of runs (whose time is then the series of two
    pieces, and whose length is found by bisection when the guess is more than one off) and outside them."""
    hws = [wl.Hardware(r * 2e12, 2e12, 900 * wl.GIB, 4e11) for r in (0.99, 0.998, 0.9995, 0.9999, 7.9, 7.98, 7.995)]
    g = wl.make_grid([wl.DENSE_70B, wl.DENSE_7B], hws, wl.Axis.table([1, 2, 7, 40]), wl.Axis.table([1]), wl.Axis.table([1]),
                     wl.Axis.table([1]), wl.Axis.table([16]), wl.Axis.table([16]), wl.Axis.table([512, 8192]))
    tr = wl.request_trace(n=80, seed=5)
    idx = np.arange(g.size, dtype=np.uint32)
    _check(torch_cuda, ora, g, idx, np.where(idx % 3, 0.2, 5.0), tr)


def test_compute_bound_lists_cost_about_as_much_as_others(torch_cuda):
    """Runs whose attention is bound by arithmetic are advanced at once like the others (step by step they took
    eight times as long as the same list on GPUs with a hundred times the peak)."""
    torch, times = torch_cuda, []
    for peak in (1e13, 1e15):
        g = wl.make_grid([wl.DENSE_70B, wl.DENSE_7B], [wl.Hardware(peak, 8e12, 900 * wl.GIB, 4e11)], wl.Axis.geom2(1, 9),
                         wl.Axis.table([1]), wl.Axis.table([1]), wl.Axis.table([1, 8]), wl.Axis.table([16, 4]),
                         wl.Axis.table([16]), wl.Axis.table([2048, 8192]))
        n = 16384
        idx = (np.arange(n) % g.size).astype(np.uint32)
        tr = wl.request_trace(n=200, seed=7)
        ctx, out = bridge.gpu_context(g), {k: torch.zeros(n, dtype=torch.float64, device="cuda") for k in guide.SIM_COLUMNS}
        ws = torch.empty(ctx.simulate_workspace_bytes(n, 200), dtype=torch.uint8, device="cuda")
        call = ctx.prepared("simulate", bridge.gpu_grid(g), torch.from_numpy(idx.view(np.int32)).cuda(),
                            torch.full((n,), 0.02, dtype=torch.float64, device="cuda"), (tr.arrival_unit, tr.n_in, tr.n_out),
                            out, ws)
        t = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            call()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        times.append(min(t))
    assert times[0] <= 3.0 * times[1], times


def test_arrival_rates_at_the_ends_of_the_range(ora, torch_cuda):
    """Rates that are divided instead of multiplied by a reciprocal: everything at once, and so far apart that a step
    does not move the clock at all (rates in between, such as 1e-9, lose the steps' low digits in the clock's: at
    4e10 s a unit in the last place is 8e-6 s, one per cent of a step, on either side of the comparison)."""
    g = wl.grid_full()
    tr = wl.request_trace(n=40, seed=11)
    idx, rate = wl.sim_configs(g, 260, seed=12)
    rate = rate.copy()
    rate[::4] = np.inf
    rate[1::4] = 1e300
    rate[2::4] = 1e-130
    _check(torch_cuda, ora, g, idx, rate, tr)


@pytest.mark.parametrize("sched", [0, 1])
def test_results_do_not_depend_on_the_list(torch_cuda, sched):
    """Which configurations share a wave differs from list to list and from call to call.  A configuration's results do
    not: bit for bit the same in a list that mixes lanes whose attention can be bound by arithmetic with lanes whose
    cannot, in that list once more, in the list backwards, and alone."""
    hws = wl.hw_profiles(3, 5) + [wl.Hardware(1e13, 8e12, 900 * wl.GIB, 4e11), wl.Hardware(3e13, 4e12, 900 * wl.GIB, 4e11)]
    g = wl.make_grid([wl.DENSE_70B, wl.DENSE_7B], hws, wl.Axis.geom2(1, 7), wl.Axis.table([1]), wl.Axis.table([1]),
                     wl.Axis.table([1, 8]), wl.Axis.table([16, 4]), wl.Axis.table([16]), wl.Axis.table([2048]))
    n = 8192
    rng = np.random.default_rng(17)
    idx = rng.integers(0, g.size, n).astype(np.uint32)
    rate = rng.choice([0.05, 0.5, 4.0], n)
    tr = wl.request_trace(n=70, seed=17)
    ctx = bridge.gpu_context(g)

    def run(pick):
        return _run(torch_cuda, ctx, g, np.ascontiguousarray(idx[pick]), np.ascontiguousarray(rate[pick]), tr, scheduler=sched)
    whole = run(np.arange(n))
    assert (whole["status"] == 0).any()
    for got, at in ((run(np.arange(n)), np.arange(n)), (run(np.arange(n)[::-1]), np.arange(n)[::-1])):
        for k in whole:
            np.testing.assert_array_equal(got[k], whole[k][at], err_msg=k)
    for c in np.linspace(0, n - 1, 40).astype(np.int64):
        alone = run(np.array([c]))
        for k in whole:
            np.testing.assert_array_equal(alone[k], whole[k][c:c + 1], err_msg=k)
