"""Performance cases: the work that a user of libguide has it do, through its public entry points.

Every case is a dict of plain values.  `kind` names the entry point:

* step      guide_eval_select: all seven columns of a grid, the cheapest configurations under a TTFT cap and the
            (TTFT, cost) front in one call -- what the optimiser does for every question it is asked
* grid      guide_eval_grid with one efficiency sample: the columns alone
* sweep     guide_eval_grid with many efficiency samples: mean / p10 / p90 columns
* extras    guide_eval_extras: cluster-level columns under a GPU budget
* sampled   guide_eval_sampled: the random-sampled space, reduced outputs (and columns when asked for)
* simulate  guide_simulate: continuous batching of a request trace
* topk      guide_select TOPK over stored columns, with or without groups
* pareto    guide_select PARETO over stored columns

`exact` is the performance model once more, in plain torch / numpy float64 from the definitions in guide.h.
"""
import math

import numpy as np
import torch

from paper_2412_04788_amd import guide, workloads as wl

DEV = "cuda"
ROOFLINE, ADDITIVE = guide.TIME_ROOFLINE, guide.TIME_ADDITIVE
AXES = ("batch", "s_in", "s_out", "tp", "wbits", "kv_block", "mbt")
INT_COLUMNS = {"b_max": torch.int32, "feasible": torch.uint8, "bucket": torch.int32, "status": torch.int32,
               "n_steps": torch.int64, "n_request_steps": torch.int64, "s_max": torch.int32, "dp_max": torch.int32,
               "max_parallelism": torch.int64, "b_adj": torch.int32, "n_sub_batches": torch.int32,
               "n_segments": torch.int32, "s_adj": torch.int32, "b_max_kept": torch.int32, "s_max_kept": torch.int32,
               "feasible_kept": torch.uint8, "feasible_count": torch.int64, "win_idx": torch.int64, "hist": torch.int64}
FRONT_CAP = 1 << 16
KV_KEEP = 0.2           # H2O's usual heavy-hitter budget


# ------------------------------------------------------------------------------------------------------ the cases

def _grid(models=5, hw=6, batch=11, s_in=10, s_out=8, tp=4, wbits=3, kv_block=2, mbt=3, odd=False, first=0, count=0):
    """Axis lengths of a grid; count = 0: the whole grid.  odd: values that are no powers of two."""
    return dict(models=models, hw=hw, batch=batch, s_in=s_in, s_out=s_out, tp=tp, wbits=wbits, kv_block=kv_block, mbt=mbt,
                odd=odd, first=first, count=count)


def listed():
    return [
        # the smallest question: one model on one GPU type, 1080 configurations -- launches and latency are all of it
        dict(name="step_tiny", kind="step", additive=False, k=3, **_grid(1, 1, 9, 6, 5, 4, 1, 1, 1)),
        # the ordinary question: five models on six GPU types, 1 900 800 configurations (the benchmark's step)
        dict(name="step_full", kind="step", additive=False, k=3, **_grid()),
        # a catalogue of 64 GPU types: 20 275 200 configurations, 912 MB of columns in one call
        dict(name="grid_large", kind="grid", additive=False, **_grid(hw=64)),
        # a study of the serving engine's own knobs: five block sizes and six token budgets, odd values, the
        # additive time model, a ragged part of the grid
        dict(name="grid_wide_axes", kind="grid", additive=True,
             **_grid(3, 4, 7, 6, 5, 3, 2, 5, 6, odd=True, first=1237, count=443_211)),
        # uncertainty of every configuration of the full grid: 64 efficiency samples each
        dict(name="sweep_full", kind="sweep", additive=False, samples=64, **_grid()),
        # cluster-level view of the full grid under a budget of 8 GPUs, all twelve columns
        dict(name="extras_full", kind="extras", additive=False, n_gpus=8, **_grid()),
        # random search: 2^28 candidates, reduced outputs only
        dict(name="sampled_full", kind="sampled", additive=False, count=1 << 28, columns=False),
        # serving simulation of 65 536 configurations x 1024 requests, every engine step stepped
        dict(name="sim_stepped", kind="simulate", additive=False, prefill_first=False, closed=False, n_cfg=65536, n_req=1024,
             **_grid()),
        # the same size under the other scheduler, runs of decode-only steps in closed form
        dict(name="sim_closed", kind="simulate", additive=False, prefill_first=True, closed=True, n_cfg=65536, n_req=1024,
             **_grid()),
        # a short list of candidates against a short trace, as after a first selection
        dict(name="sim_short", kind="simulate", additive=True, prefill_first=False, closed=False, n_cfg=1999, n_req=97,
             **_grid(3, 4, 11, 1, 1, 4, 3, 2, 3, odd=True)),
        # the top three of each of ten model-size classes over 1.9 M stored rows
        dict(name="topk_groups", kind="topk", rows=1_900_800, k=3, groups=10, constraints=1),
        # the (p90 TTFT, cost) front over stored columns of 1.9 M rows, under a cap on a third column
        dict(name="pareto_rows", kind="pareto", rows=1_900_799, constraints=1, spread=0.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_grid(rng, most):
    """Axis lengths with 1 .. most configurations, and a range of them."""
    while True:
        g = _grid(rng.randint(1, 5), _log(rng, 1, 64), rng.randint(1, 11), rng.randint(1, 10), rng.randint(1, 8),
                  rng.randint(1, 4), rng.randint(1, 3), rng.randint(1, 5), rng.randint(1, 6), odd=rng.random() < 0.5)
        size = _grid_size(g)
        if 500 <= size <= most:
            break
    if rng.random() < 0.5:
        g["first"] = rng.randrange(size // 3)
        g["count"] = rng.randint(size // 3, size - g["first"])
    return g


def draw(rng):
    kind = rng.choice(("step", "step", "grid", "sweep", "extras", "sampled", "simulate", "topk", "pareto"))
    additive = rng.random() < 0.3
    if kind == "step":
        return dict(kind=kind, additive=additive, k=rng.choice((1, 3, 4, 8)), **_draw_grid(rng, 4_000_000))
    if kind == "grid":
        return dict(kind=kind, additive=additive, **_draw_grid(rng, 20_000_000))
    if kind == "sweep":
        return dict(kind=kind, additive=additive, samples=rng.randint(2, 64), **_draw_grid(rng, 1_900_800))
    if kind == "extras":
        return dict(kind=kind, additive=additive, n_gpus=rng.choice((1, 8, 13, 64)), **_draw_grid(rng, 2_000_000))
    if kind == "sampled":
        columns = rng.random() < 0.3
        return dict(kind=kind, additive=additive, count=_log(rng, 10_000, 1 << (22 if columns else 28)), columns=columns)
    if kind == "simulate":
        return dict(kind=kind, additive=additive, prefill_first=rng.random() < 0.5, closed=rng.random() < 0.5,
                    n_cfg=_log(rng, 100, 65536), n_req=_log(rng, 16, 1024),
                    **_grid(rng.randint(1, 5), rng.randint(1, 16), 11, 1, 1, 4, 3, 2, 3, odd=rng.random() < 0.5))
    if kind == "topk":
        return dict(kind=kind, rows=_log(rng, 1000, 8_000_000), k=rng.randint(1, 8), groups=rng.choice((0, 0, 1, 10, 64)),
                    constraints=rng.randint(0, 2))
    return dict(kind=kind, rows=_log(rng, 1000, 4_000_000), constraints=rng.randint(0, 2),
                spread=rng.choice((0.1, 0.5, 1.0)))


# ------------------------------------------------------------------------------------------------------ the inputs

def _grid_size(c):
    n = c["models"] * c["hw"]
    for a in AXES:
        n *= c[a]
    return n


def _range_of(c):
    return c["first"], (c["count"] or _grid_size(c) - c["first"])


_STARTS = dict(batch=1, s_in=64, s_out=64, tp=1, wbits=None, kv_block=8, mbt=512)
_RANGES = dict(batch=(1, 1024), s_in=(64, 32768), s_out=(64, 8192), tp=(1, 16), kv_block=(8, 256), mbt=(512, 16384))


def _axes(c, seed):
    """Nine (values, geom2_start) pairs and the model / hardware records."""
    rng = np.random.Generator(np.random.PCG64([seed, 1]))
    axes = [(tuple(range(c["models"])), 0), (tuple(range(c["hw"])), 0)]
    for a in AXES:
        n = c[a]
        if a == "wbits":
            axes.append(((16, 8, 4)[:n], 0))
        elif c["odd"]:
            lo, hi = _RANGES[a]
            v = np.sort(np.rint(np.exp(rng.uniform(math.log(lo), math.log(hi), n))).astype(np.int64))
            axes.append((tuple(int(x) for x in v + np.arange(n)), 0))            # + arange: no value twice
        else:
            start = {"kv_block": 16 if n <= 2 else 8, "mbt": 2048 if n <= 3 else 512}.get(a, _STARTS[a])
            values = tuple(start << i for i in range(n))
            axes.append((values, 0 if a in ("kv_block", "mbt") else start))
    return axes, wl.MODELS_FULL[:c["models"]], wl.hw_profiles(seed, c["hw"])


def _context(models, hws):
    ctx = guide.Context(0)
    ctx.set_models(wl.models_array(models))
    ctx.set_hardware(wl.hw_array(hws))
    return ctx


def _columns(names, n):
    # zeros: what a call does not write (infeasible rows, the tail of a front) compares equal
    return {k: torch.zeros(n, dtype=INT_COLUMNS.get(k, torch.float64), device=DEV) for k in names}


def _eff(seed, n):
    return wl.efficiency_pairs(seed, n)


def _trace(c, seed):
    return wl.request_trace(seed, c["n_req"])


def _space(seed):
    s = wl.sample_space()
    d = {f: getattr(s, f) for f in ("heads", "peak", "bw", "cap", "batch", "s_in", "s_out", "tp", "wbits", "kv_block", "mbt",
                                    "kv_choices", "layers_lo", "layers_n", "ffn_lo_x2", "ffn_span_x2", "vocab", "link_div")}
    d["cap"] = np.random.Generator(np.random.PCG64([seed, 2])).permutation(d["cap"])
    return d


def _rows_data(c, seed):
    """Columns as an evaluation leaves them: latency and cost against each other over several decades, runs of equal
    neighbours, a share of infeasible rows, a third column for a cap and a class per row."""
    n = c["rows"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    run = 6
    m = -(-n // run)

    def uniform():
        return torch.rand(m, generator=gen, device=DEV, dtype=torch.float64)
    u, v = uniform(), torch.randn(m, generator=gen, device=DEV, dtype=torch.float64)
    x = torch.exp(9.0 * u - 5.0)                                               # 7 ms .. 55 s
    y = torch.exp(2.0 - 4.0 * u + c.get("spread", 0.5) * v.abs() * 4.0)        # cheaper where slower
    t3 = torch.exp(2.0 * torch.randn(m, generator=gen, device=DEV, dtype=torch.float64))
    x, y, t3 = (a.repeat_interleave(run)[:n].contiguous() for a in (x, y, t3))
    feas = (torch.rand(n, generator=gen, device=DEV) < 0.67).to(torch.uint8)
    d = dict(x=x, y=y, t3=t3, feasible=feas)
    if c.get("groups"):
        d["group"] = torch.randint(0, c["groups"], (m,), generator=gen, device=DEV, dtype=torch.int32
                                   ).repeat_interleave(run)[:n].contiguous()
    return d


def _caps(c):
    return [("x", 0.5), ("t3", 2.0)][:c["constraints"]] if c["kind"] == "topk" else [("t3", 2.0), ("x", 20.0)][:c["constraints"]]


def prepare(case, seed):
    c, kind = case, case["kind"]
    tm = ADDITIVE if c.get("additive") else ROOFLINE
    if kind in ("topk", "pareto"):
        ctx = _context(wl.MODELS_FULL[:1], [wl.HW_TINY])
        d = _rows_data(c, seed)
        cons = [(d[name], cap) for name, cap in _caps(c)]
        n = c["rows"]
        if kind == "topk":
            g = max(c["groups"], 1)
            out = dict(idx=torch.zeros(g * c["k"], dtype=torch.int64, device=DEV),
                       val=torch.zeros(g * c["k"], dtype=torch.float64, device=DEV),
                       count=torch.zeros(g, dtype=torch.int64, device=DEV))
            ws = torch.empty(ctx.select_workspace_bytes(guide.SELECT_TOPK, n, g), dtype=torch.uint8, device=DEV)
            call = ctx.prepared("select", guide.SELECT_TOPK, n, d["y"], out["idx"], out["val"], out["count"], ws,
                                feasible=d["feasible"], constraints=cons, group=d.get("group"), n_groups=g, k=c["k"])
        else:
            out = dict(idx=torch.zeros(FRONT_CAP, dtype=torch.int64, device=DEV),
                       count=torch.zeros(1, dtype=torch.int64, device=DEV))
            ws = torch.empty(ctx.select_workspace_bytes(guide.SELECT_PARETO, n), dtype=torch.uint8, device=DEV)
            call = ctx.prepared("select", guide.SELECT_PARETO, n, d["x"], out["idx"], None, out["count"], ws,
                                objective_y=d["y"], feasible=d["feasible"], constraints=cons, capacity=FRONT_CAP)
        return dict(call=call, out=out, keep=(ctx, d, ws))
    if kind == "sampled":
        ctx = _context(wl.MODELS_FULL[:1], [wl.HW_TINY])
        names = ("feasible_count", "win_val", "win_idx", "hist")
        out = {k: torch.zeros({"feasible_count": 1, "hist": wl.N_HIST_BINS}.get(k, wl.N_BUCKETS),
                              dtype=INT_COLUMNS.get(k, torch.float64), device=DEV) for k in names}
        if c["columns"]:
            out.update(_columns(("t_prefill", "t_batch", "cost", "b_max", "feasible", "bucket"), c["count"]))
        call = ctx.prepared("eval_sampled", _space(seed), seed, 0, c["count"], wl.BUCKET_EDGES, wl.TTFT_CAP_S, out,
                            time_model=tm)
        return dict(call=call, out=out, keep=(ctx,))
    axes, models, hws = _axes(c, seed)
    ctx = _context(models, hws)
    grid = guide.GridArg(axes)
    if kind == "simulate":
        tr = _trace(c, seed)
        idx, rate = _sim_list(c, seed)
        d_idx, d_rate = torch.from_numpy(idx.view(np.int32)).to(DEV), torch.from_numpy(rate).to(DEV)
        out = _columns(guide.SIM_COLUMNS, c["n_cfg"])
        ws = torch.empty(ctx.simulate_workspace_bytes(c["n_cfg"], c["n_req"]), dtype=torch.uint8, device=DEV)
        sched = (guide.SCHED_PREFILL_FIRST if c["prefill_first"] else guide.SCHED_SPLIT_FUSE) | \
                (guide.SIM_CLOSED_FORM_RUNS if c["closed"] else 0)
        call = ctx.prepared("simulate", grid, d_idx, d_rate, (tr.arrival_unit, tr.n_in, tr.n_out), out, ws, time_model=tm,
                            scheduler=sched)
        return dict(call=call, out=out, keep=(ctx, grid, d_idx, d_rate, ws))
    first, n = _range_of(c)
    if kind == "sweep":
        e_c, e_b = _eff(seed, c["samples"])
        out = _columns(guide.STATS_COLUMNS, n)
        call = ctx.prepared("eval_grid", grid, first, n, stats=out, e_c=e_c, e_b=e_b, time_model=tm)
        return dict(call=call, out=out, keep=(ctx, grid))
    if kind == "extras":
        out = _columns(guide.EXTRAS_COLUMNS, n)
        call = ctx.prepared("eval_extras", grid, first, n, c["n_gpus"], out, time_model=tm, kv_keep=KV_KEEP)
        return dict(call=call, out=out, keep=(ctx, grid))
    out = _columns(guide.METRIC_COLUMNS, n)
    if kind == "grid":
        call = ctx.prepared("eval_grid", grid, first, n, out=out, time_model=tm)
        return dict(call=call, out=out, keep=(ctx, grid))
    sel = dict(top_idx=torch.zeros(c["k"], dtype=torch.int64, device=DEV),
               top_val=torch.zeros(c["k"], dtype=torch.float64, device=DEV),
               top_count=torch.zeros(1, dtype=torch.int64, device=DEV),
               front=torch.zeros(FRONT_CAP, dtype=torch.int64, device=DEV),
               front_count=torch.zeros(1, dtype=torch.int64, device=DEV))
    sels = [ctx.column_select(guide.SELECT_TOPK, "cost", sel["top_idx"], sel["top_val"], sel["top_count"],
                              constraints=[("t_prefill", wl.TTFT_CAP_S)], k=c["k"]),
            ctx.column_select(guide.SELECT_PARETO, "t_prefill", sel["front"], None, sel["front_count"], objective_y="cost",
                              capacity=FRONT_CAP)]
    ws = torch.empty(ctx.eval_select_workspace_bytes(sels, n), dtype=torch.uint8, device=DEV)
    call = ctx.prepared("eval_select", grid, first, n, out, sels, ws, time_model=tm)
    return dict(call=call, out={**out, **sel}, keep=(ctx, grid, sels, ws))


def _sim_list(c, seed):
    """Configurations drawn from the grid, request rates cycling through the workload's."""
    rng = np.random.Generator(np.random.PCG64([seed, 3]))
    idx = rng.integers(0, _grid_size(c), size=c["n_cfg"], dtype=np.uint64).astype(np.uint32)
    rate = np.asarray(wl.SIM_RATES, dtype=np.float64)[np.arange(c["n_cfg"]) % len(wl.SIM_RATES)]
    return idx, np.ascontiguousarray(rate)


def run(state):
    state["call"]()
    return state["out"]


# ------------------------------------------------------------------------------------------- what it cannot do without

def work(case):
    c, kind = case, case["kind"]
    if kind in ("topk", "pareto"):
        cols = 8 * (1 + (kind == "pareto")) + 1 + 4 * bool(c.get("groups"))
        extra = len([1 for name, _ in _caps(c) if kind == "topk" or name != "x"])     # a cap on x reads no new column
        return dict(bytes=c["rows"] * (cols + 8 * extra), flops=c["rows"] * (1 + c["constraints"]))
    if kind == "sampled":
        # ten rounds of two 64 x 64 bit products (four 32-bit ones each) and about 150 operations of the model
        return dict(bytes=33_000 + (33 * c["count"] if c["columns"] else 0), flops=230 * c["count"])
    if kind == "simulate":
        # a request is admitted, prefilled and retired (two pass times of about 40 operations); stepped, about 112
        # decode steps of ten operations per request beside it; per configuration 4 + 8 bytes in, 52 out
        per = 80 + (0 if c["closed"] else 112 * 10)
        return dict(bytes=64 * c["n_cfg"] + 16 * c["n_req"], flops=per * c["n_cfg"] * c["n_req"])
    n = _range_of(c)[1]
    tile = c["kv_block"] * c["mbt"]
    if kind == "sweep":
        # per sample: three operations for each of seven tasks of a decode step (shared by the tile) and of up to
        # two prefill passes (shared by the block sizes)
        return dict(bytes=61 * n, flops=n * c["samples"] * (45 / c["kv_block"] + 30 / tile))
    if kind == "extras":
        return dict(bytes=65 * n, flops=n * (30 + 150 / tile))
    return dict(bytes=45 * n, flops=n * (12 + 60 / c["kv_block"] + 80 / tile))


def tolerance(case):
    kind = case["kind"]
    if kind in ("topk", "pareto"):
        return "exact"          # values are copied from the columns, rows are decided by comparing them
    if kind == "simulate":
        # up to 3.6e5 additions to one clock: 4.3e-12 seen against a step-by-step evaluation on one core
        return dict(rel=4e-12, max=2e-11)
    # sums of a few dozen terms, reciprocals instead of divisions, series in closed form: 2.5e-16 seen in the norm,
    # 3e-13 in the worst single value (a decode series summed term by term); a front may swap rows that tie in rounding
    return dict(rel=2e-15, max=1e-12, differ=1e-4 if kind == "step" else 0.0)


# ----------------------------------------------------------------------------------------------- the model in 64 bits

def _tables(axes, models, hws, first, n):
    """One tensor per quantity for rows [first, first + n) of the grid."""
    i = torch.arange(first, first + n, device=DEV, dtype=torch.int64)
    v = {}
    for name, (values, _) in reversed(list(zip(("model", "hw") + AXES, axes))):
        t = torch.tensor(values, dtype=torch.int64, device=DEV)
        v[name] = t[i % len(values)]
        i = i // len(values)
    m = torch.tensor(np.asarray(wl.models_array(models), dtype=np.float64), device=DEV)[v["model"]]
    h = torch.tensor(wl.hw_array(hws), device=DEV)[v["hw"]]
    r = {k: m[:, j] for j, k in enumerate(("L", "d", "n_h", "n_kv", "d_ff", "V", "E", "k"))}
    r.update({k: h[:, j] for j, k in enumerate(("peak", "bw", "cap", "link", "lat"))})
    r.update({k: v[a].double() for k, a in (("b", "batch"), ("s", "s_in"), ("o", "s_out"), ("p", "tp"), ("bits", "wbits"),
                                            ("blk", "kv_block"), ("mbt", "mbt"))})
    return r


def _coefficients(r, xp=torch):
    """FLOPs, weight bytes and activation bytes of the layer's tasks, per GPU."""
    d, p, w = r["d"], r["p"], r["bits"] / 8
    dh = xp.floor(d / r["n_h"])
    dq, dkv = r["n_h"] * dh, r["n_kv"] * dh
    moe = (r["E"] > 1) * 1.0
    ff, k, E = r["d_ff"], r["k"], r["E"]
    q = dict(L=r["L"], E=E, k=k, moe=moe)
    q["ops"] = [  # FLOPs per token, weight bytes, activation bytes per token, weights counted per expert
        (2 * d * (dq + 2 * dkv) / p, w * d * (dq + 2 * dkv) / p, 2 * d + 2 * (dq + 2 * dkv) / p, False),
        (2 * dq * d / p, w * dq * d / p, 2 * dq / p + 2 * d, False),
        (2 * k * 2 * d * ff / p, w * 2 * d * ff / p, 2 * d + 4 * k * ff / p, True),
        (2 * k * ff * d / p, w * ff * d / p, 2 * k * ff / p + 2 * d, True),
        (2 * d * E * moe, w * d * E * moe, (2 * d + 2 * E) * moe, False)]
    gkv = xp.ceil(r["n_kv"] / p) * dh
    q["att"] = (4 * dq / p, 4 * dq / p, 4 * gkv)
    q["norm"] = 8 * d
    q["lm"] = (2 * d * r["V"] / p, w * d * r["V"] / p, 2 * d + 2 * r["V"] / p)
    q["ar"] = (2 * (p - 1) / p * 2 * d / r["link"], 2 * (p - 1) * r["lat"])
    params = r["L"] * (2 * d * dq + 2 * d * dkv + 3 * E * d * ff + moe * d * E) + 2 * r["V"] * d
    q["params"], q["free"] = params, r["cap"] - w * params / p
    q["kv_tok"] = 2 * r["L"] * gkv * 2
    return q


def _op(additive, xp):
    return (lambda a, b: a + b) if additive else xp.maximum


def _minimum(xp, a, b):
    return xp.minimum(a, b)


def _base(q, peak, bw, T, additive, xp=torch):
    """One layer without attention."""
    op, t = _op(additive, xp), 0.0
    eld = _minimum(xp, q["E"], q["k"] * T)
    for f, w, a, experts in q["ops"]:
        t = t + op(f * T / peak, ((w * eld if experts else w) + a * T) / bw)
    return t + q["norm"] * T / bw + 2 * (q["ar"][0] * T + q["ar"][1])


def _lm(q, peak, bw, n, additive, xp=torch):
    f, w, a = q["lm"]
    return _op(additive, xp)(f * n / peak, (w + a * n) / bw) * (n > 0)


def _att(q, peak, bw, T, Q, K, additive, xp=torch):
    f, a, c = q["att"]
    return _op(additive, xp)(f * Q / peak, (a * T + c * K) / bw)


def _pass(q, peak, bw, T, Q, K, n, additive, xp=torch):
    return q["L"] * (_base(q, peak, bw, T, additive, xp) + _att(q, peak, bw, T, Q, K, additive, xp)) + \
        _lm(q, peak, bw, n, additive, xp)


def _times(r, q, additive, e_c=1.0, e_b=1.0):
    peak, bw, b, s, mbt = r["peak"] * e_c, r["bw"] * e_b, r["b"], r["s"], r["mbt"]
    # prefill: sub-batches of floor(mbt / s) prompts, the rest in one more pass
    per = torch.clamp(torch.minimum(torch.floor(mbt / s), b), min=1)
    full = torch.floor(b / per)
    rest = b - full * per
    short = full * _pass(q, peak, bw, per * s, per * s * s, per * s, per, additive)
    one = torch.clamp(rest, min=1)
    short = short + (rest > 0) * _pass(q, peak, bw, one * s, one * s * s, one * s, one, additive)
    # or ceil(s / mbt) segments per request
    n_seg = torch.ceil(s / mbt)
    long = torch.zeros_like(s)
    for j in range(int(n_seg.max())):
        c = torch.clamp(torch.minimum(s - j * mbt, mbt), min=0)
        ctx = j * mbt + c
        last = (n_seg == j + 1) * 1.0
        long = long + (c > 0) * _pass(q, peak, bw, c, c * ctx, ctx, last, additive)
    t_pre = torch.where(s <= mbt, short, b * long)
    # decode: steps j = 1 .. n at context s + j; attention is linear in the context on either side of one crossover
    n = r["o"] - 1
    f, a, c = q["att"]
    alpha, beta, gamma = f * b / peak, c * b / bw, a * b / bw

    def contexts(lo, hi):                       # sum of s + j for lo < j <= hi
        return (hi - lo) * s + (hi * (hi + 1) - lo * (lo + 1)) / 2
    zero = torch.zeros_like(n)
    if additive:
        att = (alpha + beta) * contexts(zero, n) + gamma * n
    else:
        cross = torch.where(alpha > beta, torch.floor(gamma / (alpha - beta) - s), n)
        cross = torch.minimum(torch.clamp(cross, min=0), n)
        att = beta * contexts(zero, cross) + gamma * cross + alpha * contexts(cross, n)
    t_dec = n * (q["L"] * _base(q, peak, bw, b, additive) + _lm(q, peak, bw, b, additive)) + q["L"] * att
    return t_pre, t_dec


def _whole(x):
    return torch.clamp(torch.floor(x), min=0, max=4294967295.0).to(torch.int64)


def _memory(r, q):
    kv = torch.ceil((r["s"] + r["o"]) / r["blk"]) * r["blk"] * q["kv_tok"]
    room = q["free"] > 0
    return torch.where(room, _whole(q["free"] / kv), 0), room & (r["b"] * kv <= q["free"])


def _metrics(c, seed, first, n):
    axes, models, hws = _axes(c, seed)
    parts = []
    for at in range(first, first + n, 1 << 21):
        r = _tables(axes, models, hws, at, min(1 << 21, first + n - at))
        q = _coefficients(r)
        t_pre, t_dec = _times(r, q, c["additive"])
        b_max, feas = _memory(r, q)
        t = t_pre + t_dec
        parts.append(dict(t_prefill=t_pre, t_decode=t_dec, t_batch=t,
                          decode_tok_s=torch.where(r["o"] > 1, r["b"] * (r["o"] - 1) / t_dec, 0.0),
                          cost=r["p"] * t / 3600.0 * 1e6 / (r["b"] * r["o"]), b_max=b_max.to(torch.int32),
                          feasible=feas.to(torch.uint8)))
    return {k: torch.cat([p[k] for p in parts]) for k in parts[0]}


def _sweep(c, seed):
    axes, models, hws = _axes(c, seed)
    first, n = _range_of(c)
    e_c, e_b = _eff(seed, c["samples"])
    S, parts = c["samples"], []
    for at in range(first, first + n, 1 << 19):
        r = _tables(axes, models, hws, at, min(1 << 19, first + n - at))
        q = _coefficients(r)
        pre, bat = [], []
        for j in range(S):
            t_pre, t_dec = _times(r, q, c["additive"], float(e_c[j]), float(e_b[j]))
            pre.append(t_pre)
            bat.append(t_pre + t_dec)
        p = {}
        for name, v in (("ttft", torch.stack(pre)), ("t_batch", torch.stack(bat))):
            p[name + "_mean"] = v.sum(0) / S
            v = v.sort(0).values
            p[name + "_p10"], p[name + "_p90"] = v[-(-S // 10) - 1], v[-(-9 * S // 10) - 1]
        b_max, feas = _memory(r, q)
        p.update(cost=r["p"] * p["t_batch_mean"] / 3600.0 * 1e6 / (r["b"] * r["o"]), b_max=b_max.to(torch.int32),
                 feasible=feas.to(torch.uint8))
        parts.append(p)
    return {k: torch.cat([p[k] for p in parts]) for k in parts[0]}


def _extras(c, seed):
    axes, models, hws = _axes(c, seed)
    first, n = _range_of(c)
    parts = []
    for at in range(first, first + n, 1 << 21):
        r = _tables(axes, models, hws, at, min(1 << 21, first + n - at))
        q = _coefficients(r)
        one = dict(r, p=torch.ones_like(r["p"]))
        steps = r["b"] * (r["o"] - 1)
        tok = torch.where(r["o"] > 1, steps / _times(r, q, c["additive"])[1], 0.0)
        tok1 = torch.where(r["o"] > 1, steps / _times(one, _coefficients(one), c["additive"])[1], 0.0)
        dp = torch.floor(c["n_gpus"] / r["p"])
        b_max, _ = _memory(r, q)
        room, length = q["free"] > 0, r["s"] + r["o"]
        s_max = torch.where(room, _whole(q["free"] / (r["b"] * q["kv_tok"])), 0)
        split = torch.clamp(torch.minimum(torch.floor(r["mbt"] / r["s"]), r["b"]), min=1)
        kept = torch.ceil(torch.ceil(KV_KEEP * length) / r["blk"]) * r["blk"] * q["kv_tok"]
        whole_s = torch.floor(q["free"] / (r["b"] * q["kv_tok"]))
        p = dict(s_max=s_max, dp_max=dp, max_parallelism=dp * b_max, cluster_tok_s=dp * tok,
                 paper_tok_s=dp * r["p"] * tok1 / (1 + torch.log2(r["p"])), b_adj=torch.minimum(r["b"], b_max.double()),
                 n_sub_batches=torch.where(r["s"] > r["mbt"], r["b"], torch.ceil(r["b"] / split)),
                 n_segments=torch.ceil(r["s"] / r["mbt"]), s_adj=torch.minimum(length, s_max.double()),
                 b_max_kept=torch.where(room, _whole(q["free"] / kept), 0),
                 s_max_kept=torch.where(room, _whole(whole_s / KV_KEEP), 0), feasible_kept=room & (r["b"] * kept <= q["free"]))
        parts.append({k: v.to(INT_COLUMNS.get(k, torch.float64)) for k, v in p.items()})
    return {k: torch.cat([p[k] for p in parts]) for k in parts[0]}


# Philox4x64-10 on int64 tensors (two's complement; shifts made logical with masks).
_M32 = 0xFFFFFFFF


def _signed(x):
    return x - (1 << 64) if x >= 1 << 63 else x


def _mul128(m, x):
    """(high, low) words of the constant m times x, both unsigned 64 bits."""
    m0, m1 = m & _M32, m >> 32
    x0, x1 = x & _M32, (x >> 32) & _M32

    def mul(a, b):                              # the low 64 bits of the product of two 32-bit values
        return b * _signed(a)
    p00, p01, p10, p11 = mul(m0, x0), mul(m1, x0), mul(m0, x1), mul(m1, x1)
    mid = ((p00 >> 32) & _M32) + (p01 & _M32) + (p10 & _M32)
    high = p11 + ((p01 >> 32) & _M32) + ((p10 >> 32) & _M32) + ((mid >> 32) & _M32)
    return high, x * _signed(m)


def _philox(i, seed):
    c = [i, torch.zeros_like(i), torch.zeros_like(i), torch.zeros_like(i)]
    k0, k1 = seed, 0
    for _ in range(10):
        h0, l0 = _mul128(0xD2E7470EE14C6C93, c[0])
        h1, l1 = _mul128(0xCA5A826395121157, c[2])
        c = [h1 ^ c[1] ^ _signed(k0), l1, h0 ^ c[3] ^ _signed(k1), l0]
        k0, k1 = (k0 + 0x9E3779B97F4A7C15) % (1 << 64), (k1 + 0xBB67AE8584CAA73B) % (1 << 64)
    return c


def _sampled(c, seed):
    sp = _space(seed)

    def tab(a):
        return torch.tensor(np.asarray(a, dtype=np.float64), device=DEV)
    lat = {k: tab(sp[k]) for k in ("heads", "peak", "bw", "cap", "batch", "s_in", "s_out", "tp", "wbits", "kv_block", "mbt",
                                   "kv_choices")}
    edges = torch.tensor(wl.BUCKET_EDGES, dtype=torch.float64, device=DEV)
    hist = torch.zeros(wl.N_HIST_BINS, dtype=torch.int64, device=DEV)
    n_feas = torch.zeros(1, dtype=torch.int64, device=DEV)
    win = torch.full((wl.N_BUCKETS,), math.inf, dtype=torch.float64, device=DEV)
    row = torch.full((wl.N_BUCKETS,), -1, dtype=torch.int64, device=DEV)
    cols, chunk = [], 1 << 22
    for at in range(0, c["count"], chunk):
        i = torch.arange(at, min(at + chunk, c["count"]), device=DEV, dtype=torch.int64)
        words = _philox(i, seed)
        u = [(words[j >> 2] >> (16 * (j & 3))) & 0xFFFF for j in range(14)]
        nh = lat["heads"][u[1] >> 6]
        kvc = lat["kv_choices"][u[2] >> 14]
        ratio = (sp["ffn_lo_x2"] + sp["ffn_span_x2"] * u[3].double() / 65536) / 2
        r = dict(L=(sp["layers_lo"] + ((u[0] * sp["layers_n"]) >> 16)).double(), d=128 * nh, n_h=nh,
                 n_kv=torch.where(kvc > 0, kvc, nh), d_ff=128 * torch.floor(ratio * nh + 0.5),
                 V=torch.full_like(nh, sp["vocab"]), E=torch.ones_like(nh), k=torch.ones_like(nh),
                 peak=lat["peak"][u[4] >> 6], bw=lat["bw"][u[5] >> 6], cap=lat["cap"][(u[6] * 6) >> 16],
                 b=lat["batch"][u[7] >> 6], s=lat["s_in"][u[8] >> 6], o=lat["s_out"][u[9] >> 6], p=lat["tp"][u[10] >> 14],
                 bits=lat["wbits"][(u[11] * 3) >> 16], blk=lat["kv_block"][u[12] >> 15], mbt=lat["mbt"][(u[13] * 3) >> 16])
        r["link"], r["lat"] = r["bw"] / sp["link_div"], torch.zeros_like(nh)
        q = _coefficients(r)
        t_pre, t_dec = _times(r, q, c["additive"])
        t = t_pre + t_dec
        cost = r["p"] * t / 3600.0 * 1e6 / (r["b"] * r["o"])
        b_max, feas = _memory(r, q)
        bucket = (q["params"][:, None] >= edges[None, :]).sum(1)
        bins = torch.clamp(torch.floor((t.view(torch.int64) >> 49).double()) - ((1023 - 12) << 3), 0, 255).to(torch.int64)
        hist += torch.bincount(bins[feas], minlength=wl.N_HIST_BINS)
        n_feas += feas.sum()
        ok = feas & (t_pre <= wl.TTFT_CAP_S)
        for g in range(wl.N_BUCKETS):
            v = torch.where(ok & (bucket == g), cost, math.inf)
            best, arg = v.min(0)
            if best < win[g]:
                win[g], row[g] = best, i[arg]
        if c["columns"]:
            cols.append(dict(t_prefill=t_pre, t_batch=t, cost=cost, b_max=b_max.to(torch.int32), feasible=feas.to(torch.uint8),
                             bucket=bucket.to(torch.int32)))
    out = dict(feasible_count=n_feas, win_val=win, win_idx=row, hist=hist)
    if cols:
        out.update({k: torch.cat([p[k] for p in cols]) for k in cols[0]})
    return out


def _topk(obj, ok, k):
    v = torch.where(ok & ~torch.isnan(obj), obj, math.inf)
    order = torch.sort(v, stable=True).indices[:k]
    val = torch.full((k,), math.inf, dtype=torch.float64, device=DEV)
    idx = torch.full((k,), -1, dtype=torch.int64, device=DEV)
    n = min(k, int(ok.sum()))
    val[:n], idx[:n] = v[order[:n]], order[:n]
    return idx, val


def _front(x, y, ok):
    rows = torch.nonzero(ok).reshape(-1)
    x, y = x[rows], y[rows]
    order = torch.sort(y, stable=True).indices
    order = order[torch.sort(x[order], stable=True).indices]                    # by (x, y, row)
    x, y, rows = x[order], y[order], rows[order]
    # the least y of strictly smaller x, and of the same x
    first = torch.ones_like(x, dtype=torch.bool)
    first[1:] = x[1:] != x[:-1]
    start = torch.cummax(torch.where(first, torch.arange(len(x), device=DEV), 0), 0).values
    least = torch.cummin(y, 0).values
    before = torch.where(start > 0, least[torch.clamp(start - 1, min=0)], math.inf)
    keep = (y < before) & (y == y[start])
    out = torch.zeros(FRONT_CAP, dtype=torch.int64, device=DEV)
    rows = rows[keep]
    out[:min(len(rows), FRONT_CAP)] = rows[:FRONT_CAP]
    return out, torch.tensor([len(rows)], dtype=torch.int64, device=DEV)


def _select(c, seed):
    d = _rows_data(c, seed)
    ok = d["feasible"] != 0
    for name, cap in _caps(c):
        ok = ok & (d[name] <= cap)
    if c["kind"] == "pareto":
        idx, count = _front(d["x"], d["y"], ok)
        return dict(idx=idx, count=count)
    picks = [ok & (d["group"] == g) for g in range(c["groups"])] if c["groups"] else [ok]
    best = [_topk(d["y"], m, c["k"]) for m in picks]
    return dict(idx=torch.cat([b[0] for b in best]), val=torch.cat([b[1] for b in best]),
                count=torch.stack([m.sum() for m in picks]))


def _simulate(c, seed):
    """The scheduler of guide.h, all configurations one engine step at a time."""
    axes, models, hws = _axes(c, seed)
    tr, (idx, rate) = _trace(c, seed), _sim_list(c, seed)
    n, m = c["n_req"], c["n_cfg"]
    v, i = {}, idx.astype(np.int64)
    for name, (values, _) in reversed(list(zip(("model", "hw") + AXES, axes))):
        v[name] = np.asarray(values, dtype=np.int64)[i % len(values)]
        i = i // len(values)
    md, hw = np.asarray(wl.models_array(models), dtype=np.float64)[v["model"]], wl.hw_array(hws)[v["hw"]]
    r = {k: md[:, j] for j, k in enumerate(("L", "d", "n_h", "n_kv", "d_ff", "V", "E", "k"))}
    r.update({k: hw[:, j] for j, k in enumerate(("peak", "bw", "cap", "link", "lat"))})
    r.update(p=v["tp"].astype(float), bits=v["wbits"].astype(float))
    q = _coefficients(r, np)
    blk, cap, mbt = v["kv_block"], v["batch"], v["mbt"]
    with np.errstate(all="ignore"):
        pool = np.where(q["free"] > 0, np.floor(q["free"] / (blk * q["kv_tok"])), 0).astype(np.int64)
    n_in, n_out = tr.n_in.astype(np.int64), tr.n_out.astype(np.int64)
    need = -(-(n_in + n_out)[None, :] // blk[:, None])
    arrive = tr.arrival_unit[None, :] / rate[:, None]
    fits = (q["free"] > 0) & (need.max(1) <= pool)
    first, fin = np.full((m, n), np.inf), np.full((m, n), np.inf)
    steps, work_done = np.zeros(m, np.int64), np.zeros(m, np.int64)
    # the state of the lanes that still run
    lane = np.nonzero(fits)[0]

    def cut(keep):
        nonlocal lane, st, Q, hwv
        lane = lane[keep]
        st = {k: a[keep] for k, a in st.items()}
        Q = {k: ([tuple(x[keep] if isinstance(x, np.ndarray) else x for x in o) for o in a] if k == "ops" else
                 tuple(x[keep] for x in a) if isinstance(a, tuple) else a[keep]) for k, a in Q.items()}
        hwv = [x[keep] for x in hwv]
    z = np.zeros(m, np.int64)
    st = dict(nx=z, head=z, part=z, dec=z, ctx=z, ds=z, done=z, free=pool, now=np.zeros(m), soon=np.full(m, 1 << 60))
    Q, hwv, lane = q, [r["peak"], r["bw"], cap, mbt], np.arange(m)
    cut(fits)
    ends = np.full((m, n), 1 << 60)
    add = c["additive"]
    while len(lane):
        nx, head, part, dec, ctx, ds, done, free, now, soon = (st[k].copy() for k in
                                                               ("nx", "head", "part", "dec", "ctx", "ds", "done", "free", "now", "soon"))
        peak, bw, cp, budget_of = hwv
        act = nx - head + dec
        jump = (act == 0) & (nx < n)
        if jump.any():
            j = np.nonzero(jump)[0]
            now[j] = np.maximum(now[j], arrive[lane[j], nx[j]])
        while True:
            can = (nx < n) & (act < cp)
            j = np.nonzero(can)[0]
            j = j[(arrive[lane[j], nx[j]] <= now[j]) & (need[lane[j], nx[j]] <= free[j])]
            if not len(j):
                break
            free[j] -= need[lane[j], nx[j]]
            nx[j] += 1
            act[j] += 1
        waits = head < nx
        run_dec = ~waits if c["prefill_first"] else np.ones(len(lane), bool)
        T = np.where(run_dec, dec, 0).astype(float)
        Qp = np.where(run_dec, ctx, 0).astype(float)
        K, lm = Qp.copy(), T.copy()
        h, prt, chunks, full = head.copy(), part.copy(), np.zeros(len(lane), np.int64), []
        left = budget_of - (0 if c["prefill_first"] else dec)
        j = np.nonzero(waits)[0]
        while len(j):
            if c["prefill_first"]:
                j = j[(chunks[j] == 0) | (n_in[np.minimum(h[j], n - 1)] <= left[j])]
            else:
                j = j[left[j] > 0]
            if not len(j):
                break
            todo = n_in[h[j]] - prt[j]
            ch = todo if c["prefill_first"] else np.minimum(todo, left[j])
            left[j] -= ch
            at = prt[j] + ch
            T[j] += ch
            Qp[j] += ch * at.astype(float)
            K[j] += at
            chunks[j] += 1
            end = ch == todo
            lm[j] += end
            e = j[end]
            full.append((e, h[e].copy()))
            h[e] += 1
            prt[j] = np.where(end, 0, at)
            j = j[h[j] < nx[j]]
        now = now + _pass(Q, peak, bw, T, Qp, K, lm, add, np)
        steps[lane] += 1
        work_done[lane] += np.where(run_dec, dec, 0) + chunks
        ds = ds + run_dec
        ctx = ctx + np.where(run_dec, dec, 0)
        j = np.nonzero(run_dec & (soon == ds))[0]
        if len(j):
            a, b = np.nonzero(ends[lane[j]] == ds[j][:, None])
            w = j[a]
            fin[lane[w], b] = now[w]
            ends[lane[w], b] = 1 << 60
            np.add.at(free, w, need[lane[w], b])
            np.add.at(dec, w, -1)
            np.add.at(done, w, 1)
            np.add.at(ctx, w, -(n_in[b] + n_out[b]))
            soon[j] = ends[lane[j]].min(1)
        for e, q_ in full:
            first[lane[e], q_] = now[e]
            short = n_out[q_] == 1
            s, t = e[short], q_[short]
            fin[lane[s], t] = now[s]
            free[s] += need[lane[s], t]
            done[s] += 1
            s, t = e[~short], q_[~short]
            dec[s] += 1
            ctx[s] += n_in[t] + 1
            ends[lane[s], t] = ds[s] + n_out[t] - 1
            soon[s] = np.minimum(soon[s], ends[lane[s], t])
        st = dict(nx=nx, head=h, part=prt, dec=dec, ctx=ctx, ds=ds, done=done, free=free, now=now, soon=soon)
        if (done >= n).any():
            cut(done < n)
    with np.errstate(all="ignore"):
        ttft = np.sort(first - arrive, axis=1)
        many = n_out > 1
        tpot = ((fin - first) / np.maximum(n_out - 1, 1))[:, many].mean(1) if many.any() else np.zeros(m)
        rate_out = n_out.sum() / (fin.max(1) - arrive[:, 0])
    bad = ~fits
    out = dict(ttft_p50=ttft[:, (n + 1) // 2 - 1], ttft_p99=ttft[:, -(-99 * n // 100) - 1], mean_tpot=tpot, tokens_s=rate_out)
    for k in out:
        out[k] = np.where(bad, 0.0 if k == "tokens_s" else np.inf, out[k])
    return dict(out, status=bad.astype(np.int32), n_steps=steps, n_request_steps=work_done)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("topk", "pareto"):
        return _select(c, seed)
    if kind == "simulate":
        # stepping many configurations through a long trace takes minutes
        return _simulate(c, seed) if c["n_cfg"] <= 4096 and c["n_req"] <= 128 else None
    if kind == "sampled":
        return _sampled(c, seed)
    if kind == "sweep":
        return _sweep(c, seed)
    if kind == "extras":
        return _extras(c, seed)
    first, n = _range_of(c)
    out = _metrics(c, seed, first, n)
    if kind == "step":
        feas = out["feasible"] != 0
        ok = feas & (out["t_prefill"] <= wl.TTFT_CAP_S)
        idx, val = _topk(out["cost"], ok, c["k"])
        front, count = _front(out["t_prefill"], out["cost"], feas)
        out.update(top_idx=idx, top_val=val, top_count=ok.sum().reshape(1), front=front, front_count=count)
    return out
