// Grid evaluation kernels: flat index -> mixed-radix digits -> candidate ->
// metrics, one candidate per lane, spec tables staged in LDS, coalesced
// structure-of-arrays stores.
#include <hip/hip_ext.h>

#include "kernels.hpp"
#include "perf_model.hpp"
#include "select_shared.hpp"

namespace guide {

// The next number of a loop that strides over 0 .. n - 1, n (the end) when there is none: i + stride may pass 2^32 near the
// largest grids, and a loop that compares the wrapped sum would start over and never end.
__device__ inline uint32_t stride_on(uint32_t i, uint32_t stride, uint32_t n) { return n - i > stride ? i + stride : n; }

struct GridLds {
    uint32_t axis[kNumAxes][GUIDE_MAX_AXIS_VALUES];
    guide_model models[GUIDE_MAX_MODELS];
    HwRecip hw[GUIDE_MAX_HW];
};

__device__ inline void stage_grid_tables(GridLds &s, const GridDesc &g, const DevTables *__restrict__ tab) {
    for (uint32_t i = threadIdx.x; i < kNumAxes * GUIDE_MAX_AXIS_VALUES; i += blockDim.x)
        (&s.axis[0][0])[i] = (&tab->axis_vals[0][0])[i];
    for (uint32_t i = threadIdx.x; i < g.n_models * 8u; i += blockDim.x)
        ((uint32_t *)s.models)[i] = ((const uint32_t *)tab->models)[i];
    for (uint32_t i = threadIdx.x; i < g.n_hw; i += blockDim.x) {
        const guide_hw h = tab->hw[i];
        HwRecip r;
        r.r_peak = 1.0 / h.peak_flops;
        r.r_bw = 1.0 / h.hbm_bw;
        r.cap = h.cap_bytes;
        r.r_link = 1.0 / h.link_bw;
        r.lat = h.link_lat;
        s.hw[i] = r;
    }
}

struct Candidate {
    uint32_t model, hw;
    Knobs kn;
};

__device__ inline Candidate decode_index(const GridLds &s, const GridDesc &g, uint32_t idx) {
    uint32_t v[kNumAxes];
    uint32_t rem = idx;
#pragma unroll
    for (int a = kNumAxes - 1; a > 0; --a) {
        const uint32_t q = div32(rem, g.div[a]);
        v[a] = s.axis[a][rem - q * g.div[a].d];
        rem = q;
    }
    v[0] = s.axis[0][rem];
    Candidate c;
    c.model = v[AX_MODEL];
    c.hw = v[AX_HW];
    c.kn.b = v[AX_BATCH];
    c.kn.s_in = v[AX_SIN];
    c.kn.s_out = v[AX_SOUT];
    c.kn.p = v[AX_TP];
    c.kn.wbits = v[AX_WBITS];
    c.kn.blk = v[AX_BLK];
    c.kn.mbt = v[AX_MBT];
    return c;
}

// GPU-hours per million generated tokens.
__device__ inline double cost_of(const Knobs &kn, double t_batch) {
    return (double)kn.p * t_batch / 3600.0 * 1.0e6 / ((double)kn.b * (double)kn.s_out);
}

// ---------------------------------------------------------------- tiled variant
//
// The two fastest axes (KV block, max batched tokens) change only part of the
// model: the decode series does not depend on either, the prefill only on the
// token budget, the memory check only on the block size.  A lane therefore takes
// one *tile* = all NB x NM combinations of those two axes for one setting of the
// seven slower axes (NB*NM consecutive flat indices), evaluates the shared parts
// once, and the wave transposes each output column through LDS so that global
// stores stay coalesced (lane l stores index base + 64*it + l).

// What a block needs besides the index range is the same for every block and every call on an
// unchanged grid: the axis values, models and hardware reciprocals, the nudged reciprocals of the
// divisors, and the per-op FLOPs / bytes of every (model, tp, precision) combination.  A one-block
// kernel derives them once into device memory (when the context's tables change); the evaluation
// blocks copy them into LDS.
constexpr uint32_t kCoefRows = 96;          // (model, tp, precision) rows of per-op coefficients kept in LDS
struct alignas(16) TileLds {
    GridLds g;
    double r_tp[GUIDE_MAX_AXIS_VALUES];     // 1 / tp
    double r_sin[GUIDE_MAX_AXIS_VALUES];    // nudged reciprocals for exact floor division
    double r_blk[GUIDE_MAX_AXIS_VALUES];
    double r_mbt[GUIDE_MAX_AXIS_VALUES];
    Coef coef[kCoefRows];                   // last: only the rows in use are copied
};
static_assert(offsetof(TileLds, coef) % 16 == 0 && sizeof(TileLds) % 16 == 0, "copied in 16-byte words");

__global__ __launch_bounds__(kBlock) void tile_tables_kernel(GridDesc g, const DevTables *__restrict__ tab,
                                                             TileLds *__restrict__ dst) {
    stage_grid_tables(dst->g, g, tab);
    for (uint32_t i = threadIdx.x; i < GUIDE_MAX_AXIS_VALUES; i += blockDim.x) {
        dst->r_tp[i] = 1.0 / (double)max(tab->axis_vals[AX_TP][i], 1u);
        dst->r_sin[i] = recip_up(1.0 / (double)max(tab->axis_vals[AX_SIN][i], 1u));
        dst->r_blk[i] = recip_up(1.0 / (double)max(tab->axis_vals[AX_BLK][i], 1u));
        dst->r_mbt[i] = recip_up(1.0 / (double)max(tab->axis_vals[AX_MBT][i], 1u));
    }
    const uint32_t n_tp = g.div[AX_TP].d, n_w = g.div[AX_WBITS].d;
    const uint32_t n_rows = g.div[AX_MODEL].d * n_tp * n_w;
    if (n_rows <= kCoefRows) {
        for (uint32_t r = threadIdx.x; r < n_rows; r += blockDim.x) {
            const uint32_t dw = r % n_w, dt = (r / n_w) % n_tp, dm = r / (n_w * n_tp);
            const uint32_t p = tab->axis_vals[AX_TP][dt];
            dst->coef[r] = make_coef(tab->models[tab->axis_vals[AX_MODEL][dm]], p, tab->axis_vals[AX_WBITS][dw],
                                     1.0 / (double)p);
        }
    }
}

// Row sample for a Pareto selection over the rows being evaluated, taken by extra blocks of the evaluation kernel
// (block `rb` of them; kBlock samples each): sample_number / sample_row give the rows.  The
// sampled rows are evaluated here from scratch rather than read back, so the sample does not wait for the columns.
// It fixes the range of x that the selection's bins slice (any range is correct, a good one is fast), and the
// block hands the front of its sample rows to the selection's filter pass (store_sample_front).
// Also resets the counters that the selection's kernels accumulate into.
constexpr uint64_t kSampleMargin = 1ull << 26;      // in key units: 2^-26 relative for a normal number
template <bool ADDITIVE>
__device__ inline void sample_rider(const GridLds &s, const GridDesc &g, uint32_t rb, uint32_t n_rider_blocks, uint32_t first,
                                    uint32_t count, double re_c, double re_b, const FusedSelect &fs) {
    constexpr int kWaves = kBlock / kWave;
    __shared__ uint64_t s_lo[kWaves];
    __shared__ Pair s_best[kWaves];
    SelectScratch *sc = (SelectScratch *)fs.scratch;
    const uint32_t gid = rb * kBlock + threadIdx.x;
    const uint32_t n_samples = n_rider_blocks * kBlock;
    if (gid == 0) sc->counters[0] = sc->counters[1] = 0;
    const uint32_t stride = count > n_samples ? count / n_samples : 1;
    const uint32_t k = sample_number(rb, n_rider_blocks);
    uint64_t lo = kNone, kx = 0, ky = 0;
    Pair best = {kNone, kNone};
    bool pass = false;
    if ((uint64_t)k * stride < count) {
        const Candidate c = decode_index(s, g, first + sample_row(k, stride));
        const Coef cf = make_coef(s.models[c.model], c.kn.p, c.kn.wbits);
        const HwRecip hw = s.hw[c.hw];
        const TimeCoef tc = make_time_coef(cf, hw.r_peak * re_c, hw.r_bw * re_b, hw.r_link, hw.lat);
        const EvalResult r = evaluate_times<ADDITIVE>(tc, c.kn);
        const double t_batch = r.t_prefill + r.t_decode;
        const double tok_s = c.kn.s_out > 1 ? (double)c.kn.b * (double)(c.kn.s_out - 1) / r.t_decode : 0.0;
        const double cost = cost_of(c.kn, t_batch);
        auto col = [&](uint32_t id) {
            return id == GUIDE_COL_T_PREFILL ? r.t_prefill
                   : id == GUIDE_COL_T_DECODE ? r.t_decode
                   : id == GUIDE_COL_T_BATCH ? t_batch
                   : id == GUIDE_COL_DECODE_TOK_S ? tok_s : cost;
        };
        // The values here come from another instruction sequence than the stored columns and may differ
        // from them in the last bits (every sequence is within 1e-9 relative of the definition), while a
        // sample row may only prune rows that the stored row dominates.  So the sample row is moved up by
        // 2^-26 relative in x and y (a point that the stored row dominates prunes no row wrongly), and it
        // must pass its filter by the same margin (a row that is not a passing row must prune nothing).
        const double x = col(fs.pareto_x), y = col(fs.pareto_y);
        bool ok = x == x && y == y;
        for (uint32_t q = 0; q < fs.pareto_filter.n_con; ++q) {
            const double v = col(fs.pareto_filter.col[q]), cap = fs.pareto_filter.cap[q];
            ok = ok && v == v && cap == cap && key_of(v) + kSampleMargin <= key_of(cap);
        }
        if (ok && fs.pareto_filter.use_feasible) {
            const double c_avail = hw.cap - cf.w_gpu;
            const uint32_t tok_req = (c.kn.s_in + c.kn.s_out + c.kn.blk - 1) / c.kn.blk * c.kn.blk;
            ok = c_avail > 0.0 && (double)c.kn.b * ((double)tok_req * cf.kv_tok) * (1.0 + 0x1p-26) <= c_avail;
        }
        if (ok) {
            pass = true;
            lo = kx = key_of(x);
            ky = key_of(y);
            best = Pair{ky, kx};
        }
    }
    lo = wave_min(lo);
    best = wave_min(best);
    if (threadIdx.x % kWave == 0) {
        s_lo[threadIdx.x / kWave] = lo;
        s_best[threadIdx.x / kWave] = best;
    }
    store_sample_front(pass, kx + kSampleMargin, ky + kSampleMargin, sc->sample_front + rb * kSampleFrontPer);
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int wv = 1; wv < kWaves; ++wv) {
            lo = min_u64(lo, s_lo[wv]);
            best = pair_min(best, s_best[wv]);
        }
        sc->sample_lo[rb] = lo;
        sc->sample_best[rb] = best;
    }
}

// FUSED: a top-k folded in (FusedSelect); every block then writes its top-K partials, also when it owns no tile.
// STREAM: full waves store the 8-byte columns with the streaming hint.
template <bool ADDITIVE, int NB, int NM, bool FUSED, bool STREAM>
__global__ __launch_bounds__(kBlock) void eval_tile_kernel(GridDesc g, const DevTables *__restrict__ tab,
                                                           uint32_t first, uint32_t count, double re_c, double re_b,
                                                           guide_metrics out, FusedSelect fs,
                                                           const TileLds *__restrict__ derived) {
    constexpr int TS = NB * NM;
    constexpr int kWaves = kBlock / kWave;
    __shared__ TileLds s;
    __shared__ double s_x[kWaves][kWave * TS];
    const uint32_t n_tp = g.div[AX_TP].d, n_w = g.div[AX_WBITS].d;
    const uint32_t n_rows = g.div[AX_MODEL].d * n_tp * n_w;
    const bool coef_in_lds = n_rows <= kCoefRows;
    {
        // every load is issued before the first LDS write, so the copy costs one memory latency
        const uint32_t vecs = (uint32_t)(offsetof(TileLds, coef) + (coef_in_lds ? n_rows : 0u) * sizeof(Coef) + 15) / 16;
        constexpr uint32_t kPer = (sizeof(TileLds) / 16 + kBlock - 1) / kBlock;
        const uint4 *src = (const uint4 *)derived;
        uint4 *dst = (uint4 *)&s;
        uint4 t[kPer];
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            const uint32_t i = q * kBlock + threadIdx.x;
            t[q] = i < vecs ? src[i] : uint4{0, 0, 0, 0};
        }
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            const uint32_t i = q * kBlock + threadIdx.x;
            if (i < vecs) dst[i] = t[q];
        }
    }
    TopList<kFusedTopK> top;
    uint64_t n_pass = 0, top_bound = kNone;
    uint32_t batch = 0;
    if (FUSED) top.init();
    __syncthreads();
    if (fs.rider_blocks && blockIdx.x >= gridDim.x - fs.rider_blocks) {                // block-uniform
        sample_rider<ADDITIVE>(s.g, g, blockIdx.x - (gridDim.x - fs.rider_blocks), fs.rider_blocks, first, count, re_c,
                               re_b, fs);
        return;
    }
    const uint32_t n_main_blocks = gridDim.x - fs.rider_blocks;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    double *xw = s_x[wave];
    const uint32_t t_first = first / TS;
    const uint32_t n_tiles = (first + count - 1) / TS - t_first + 1;
    const uint32_t last = first + count;                       // exclusive; count > 0, no overflow (grid < 2^32)
    for (uint32_t tb = (blockIdx.x * kWaves + wave) * kWave; tb < n_tiles; tb = stride_on(tb, n_main_blocks * kWaves * kWave, n_tiles)) {
        const uint32_t left = n_tiles - tb;
        const uint32_t tl = (uint32_t)lane < left ? tb + lane : n_tiles - 1;   // idle lanes repeat the last tile
        // digits of the seven slow axes
        uint32_t dg[AX_BLK];
        uint32_t rem = t_first + tl;
#pragma unroll
        for (int a = AX_BLK - 1; a > 0; --a) {
            const uint32_t q = div32(rem, g.div[a]);
            dg[a] = rem - q * g.div[a].d;
            rem = q;
        }
        dg[0] = rem;
        Knobs kn;
        kn.b = s.g.axis[AX_BATCH][dg[AX_BATCH]];
        kn.s_in = s.g.axis[AX_SIN][dg[AX_SIN]];
        kn.s_out = s.g.axis[AX_SOUT][dg[AX_SOUT]];
        kn.p = s.g.axis[AX_TP][dg[AX_TP]];
        kn.wbits = s.g.axis[AX_WBITS][dg[AX_WBITS]];
        const Coef cf = coef_in_lds
                            ? s.coef[(dg[AX_MODEL] * n_tp + dg[AX_TP]) * n_w + dg[AX_WBITS]]
                            : make_coef(s.g.models[s.g.axis[AX_MODEL][dg[AX_MODEL]]], kn.p, kn.wbits, s.r_tp[dg[AX_TP]]);
        const HwRecip hw = s.g.hw[s.g.axis[AX_HW][dg[AX_HW]]];
        const TimeCoef tc = make_time_coef(cf, hw.r_peak * re_c, hw.r_bw * re_b, hw.r_link, hw.lat);

        // coalesced stores: element e of the wave's 64*TS consecutive indices sits in lane e / TS, slot e % TS.
        // Columns leave as soon as their values exist so that stores overlap the remaining arithmetic.
        const uint32_t cfg0 = (t_first + tb) * TS;             // flat index of the wave's first element
        // every element of the wave inside [first, last): no per-element checks (wave-uniform)
        const bool full = left >= (uint32_t)kWave && cfg0 >= first && cfg0 + kWave * TS <= last;
        auto store_f64 = [&](double *col, auto value_of_slot) {
            if (!col) return;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int j = 0; j < TS; ++j) xw[lane * TS + j] = value_of_slot(j);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (full) {
                double *dst = col + (cfg0 - first) + lane;
#pragma unroll
                for (int it = 0; it < TS; ++it) {
                    if (STREAM) __builtin_nontemporal_store(xw[it * kWave + lane], &dst[it * kWave]);
                    else dst[it * kWave] = xw[it * kWave + lane];
                }
            } else {
#pragma unroll
                for (int it = 0; it < TS; ++it) {
                    const uint32_t cfg = cfg0 + it * kWave + lane;
                    const double v = xw[it * kWave + lane];
                    if (cfg >= first && cfg < last && (uint32_t)((it * kWave + lane) / TS) < left) col[cfg - first] = v;
                }
            }
        };

        // memory check: depends on the block size only
        MemResult mem[NB];
        const bool need_mem = out.b_max || out.feasible ||
                              (FUSED && fs.topk && fs.topk_filter.use_feasible);
        if (need_mem) {
            const double c_avail = hw.cap - cf.w_gpu;
            const uint32_t tok = kn.s_in + kn.s_out;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const uint32_t blk = s.g.axis[AX_BLK][k];
                const uint32_t tok_req = floor_div(tok + blk - 1, s.r_blk[k]) * blk;
                const double kv_req = (double)tok_req * cf.kv_tok;
                const double q = floor(c_avail / kv_req);
                const bool room = c_avail > 0.0;
                mem[k].feasible = room && (double)kn.b * kv_req <= c_avail;
                mem[k].b_max = !room ? 0u : (q >= 4294967295.0 ? 4294967295u : (uint32_t)q);
            }
        }
        if (out.b_max || out.feasible) {
            uint32_t *xi = (uint32_t *)xw;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int j = 0; j < TS; ++j) {
                xi[lane * TS + j] = mem[j / NM].b_max;
                xi[kWave * TS + lane * TS + j] = mem[j / NM].feasible ? 1u : 0u;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int it = 0; it < TS; ++it) {
                const uint32_t cfg = cfg0 + it * kWave + lane;
                const uint32_t bm = xi[it * kWave + lane], fe = xi[kWave * TS + it * kWave + lane];
                if (full || (cfg >= first && cfg < last && (uint32_t)((it * kWave + lane) / TS) < left)) {
                    if (out.b_max) out.b_max[cfg - first] = bm;
                    if (out.feasible) out.feasible[cfg - first] = (uint8_t)fe;
                }
            }
        }

        // decode series: depends on neither tile axis
        const double t_decode = decode_time_fast<ADDITIVE>(tc, kn.b, kn.s_in, kn.s_out - 1);
        const double tok_s = kn.s_out > 1 ? (double)kn.b * (double)(kn.s_out - 1) * fast_recip(t_decode) : 0.0;
        store_f64(out.t_decode, [&](int) { return t_decode; });
        store_f64(out.decode_tok_s, [&](int) { return tok_s; });

        // prefill: depends on the token budget only
        double t_prefill[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m)
            t_prefill[m] = prefill_time_fast<ADDITIVE>(tc, kn.b, kn.s_in, s.g.axis[AX_MBT][m], s.r_sin[dg[AX_SIN]],
                                                        s.r_mbt[m]);
        const double bs = (double)kn.b * (double)kn.s_out;
        const double cost_f = (double)kn.p * (1.0e6 / 3600.0) * fast_recip(bs);
        double t_batch[NM], cost[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            t_batch[m] = t_prefill[m] + t_decode;
            cost[m] = t_batch[m] * cost_f;
        }
        store_f64(out.t_prefill, [&](int j) { return t_prefill[j % NM]; });
        store_f64(out.t_batch, [&](int j) { return t_batch[j % NM]; });
        store_f64(out.cost, [&](int j) { return cost[j % NM]; });

        if (FUSED) {
            // The selections see exactly the values stored above.  A column's value depends on the
            // token-budget digit m at most and feasibility on the block-size digit k only, so the
            // filters and keys are worked out once per m and each row costs a few compares.
            const bool tile_real = (uint32_t)lane < left;
            const uint32_t row0 = (t_first + tl) * TS;
            auto col = [&](uint32_t id, int m) {
                return id == GUIDE_COL_T_PREFILL ? t_prefill[m]
                       : id == GUIDE_COL_T_DECODE ? t_decode
                       : id == GUIDE_COL_T_BATCH ? t_batch[m]
                       : id == GUIDE_COL_DECODE_TOK_S ? tok_s : cost[m];
            };
            auto passes = [&](const FusedFilter &f, int m) {
                bool ok = true;
                for (uint32_t c = 0; c < f.n_con; ++c) ok = ok && (col(f.col[c], m) <= f.cap[c]);
                return ok;
            };
            if (fs.topk) {
                uint64_t key[NM];
                bool ok_m[NM], cand = false;
                uint32_t n_ok = 0;
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    const double v = col(fs.topk_obj, m);
                    key[m] = key_of(v);
                    ok_m[m] = tile_real && v == v && passes(fs.topk_filter, m);
                    n_ok += ok_m[m] ? 1u : 0u;
                    cand = cand || (ok_m[m] && key[m] <= top_bound);
                }
                auto feas = [&](int k) { return !fs.topk_filter.use_feasible || mem[k].feasible; };
                if (full) {
                    // every row of the wave's tiles is in range: passing rows are counted per tile, and the
                    // rows are visited only when one of them can still enter the list
                    uint32_t n_f = 0;
#pragma unroll
                    for (int k = 0; k < NB; ++k) n_f += feas(k) ? 1u : 0u;
                    n_pass += n_ok * n_f;
                    if (cand) {
#pragma unroll
                        for (int j = 0; j < TS; ++j) {
                            const int k = j / NM, m = j % NM;
                            if (ok_m[m] && feas(k) && key[m] <= top_bound)
                                top.insert_ascending(Pair{key[m], (uint64_t)(row0 + j - first)});
                        }
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < TS; ++j) {
                        const int k = j / NM, m = j % NM;
                        const uint32_t row = row0 + j;
                        if (ok_m[m] && row >= first && row < last && feas(k)) {
                            ++n_pass;
                            if (key[m] <= top_bound) top.insert_ascending(Pair{key[m], (uint64_t)(row - first)});
                        }
                    }
                }
                // Some lane already holds K keys at or below the least K-th key of the wave's lanes, so a
                // row above it cannot be among the block's K least.  The bound tightens fast at first and
                // slowly later: refreshed after each of the first four batches, then after every fourth.
                if (batch < 4 || (batch & 3) == 0) top_bound = wave_min(top.v[kFusedTopK - 1].key);
                ++batch;
            }
        }
    }
    if (FUSED) {
        constexpr int kCap = 8;
        __shared__ Pair s_pairs[kWaves][kFusedTopK], s_cand[kWaves][kCap];
        __shared__ uint32_t s_n[kWaves];
        __shared__ uint64_t s_cnt[kWaves];
        if (fs.topk) {
            const Top1Ws w = top1_ws(fs.topk_ws);
            for (int off = kWave / 2; off > 0; off >>= 1) n_pass += __shfl_xor(n_pass, off, kWave);
            if (lane == 0) s_cnt[wave] = n_pass;
            top_bound = wave_min(top.v[kFusedTopK - 1].key);
            block_topk_bounded<kFusedTopK, kWaves, kCap>(top, top_bound, s_cand, s_n, s_pairs, [&](int r, const Pair &p) {
                w.key[(size_t)blockIdx.x * kFusedTopK + r] = p.key;
                w.idx[(size_t)blockIdx.x * kFusedTopK + r] = p.idx;
            });                                          // (contains the barrier that publishes s_cnt)
            if (threadIdx.x == 0) {
                uint64_t c = 0;
                for (int wv = 0; wv < kWaves; ++wv) c += s_cnt[wv];
                w.cnt[blockIdx.x] = c;
            }
        }
    }
}

// The R smallest (LARGEST: largest) values seen, kept sorted with the extreme one first; R <= 7 covers the
// nearest-rank p10 / p90 of up to 64 samples.  Values arrive eight at a time, already sorted ascending
// (merge), or one by one (push).  Compare-exchanges are a minimum and a maximum.
constexpr int kRankMax = 7;
constexpr int kSweepGroup = 8;
template <bool LARGEST>
struct ExtremeK {
    double v[kRankMax];
    // puts the value that belongs nearer the front of the list into a
    static __device__ void cx(double &a, double &b) {
        const double lo = fmin(a, b), hi = fmax(a, b);
        a = LARGEST ? hi : lo;
        b = LARGEST ? lo : hi;
    }
    __device__ void init() {
#pragma unroll
        for (int i = 0; i < kRankMax; ++i) v[i] = LARGEST ? -INFINITY : INFINITY;
    }
    __device__ void push(double x) {
#pragma unroll
        for (int i = 0; i < kRankMax; ++i) cx(v[i], x);
    }
    // a[0] <= ... <= a[7].  Entry i of the list meets the i-th candidate from the other end of the group's seven
    // best (the eighth cannot be among the seven best of the union): the better of each pair are the union's
    // seven best, in a sequence that rises and falls once, which the last three stages of a bitonic sorter of
    // eight put in order (its first element would be a sentinel that no exchange moves, so those are left out).
    __device__ void merge(const double (&a)[kSweepGroup]) {
        double w[kSweepGroup];
#pragma unroll
        for (int i = 0; i < kRankMax; ++i) {
            const double c = LARGEST ? a[1 + i] : a[kRankMax - 1 - i];
            w[1 + i] = LARGEST ? fmax(v[i], c) : fmin(v[i], c);
        }
        cx(w[1], w[5]); cx(w[2], w[6]); cx(w[3], w[7]);
        cx(w[1], w[3]); cx(w[4], w[6]); cx(w[5], w[7]);
        cx(w[2], w[3]); cx(w[4], w[5]); cx(w[6], w[7]);
#pragma unroll
        for (int i = 0; i < kRankMax; ++i) v[i] = w[1 + i];
    }
    // r-th from the extreme end, 0-based: the least extreme of the first r + 1.  (A chain of selects r == i ? v[i] : x
    // is turned into an indexed read, which puts the list into scratch memory.)
    __device__ double at(uint32_t r) const {
        double x = v[0];
#pragma unroll
        for (int i = 1; i < kRankMax; ++i) {
            const double y = LARGEST ? fmin(x, v[i]) : fmax(x, v[i]);
            x = (uint32_t)i <= r ? y : x;
        }
        return x;
    }
};
// Eight values in ascending order (19 compare-exchanges).
__device__ inline void sort_group(double (&a)[kSweepGroup]) {
    auto cx = [](double &x, double &y) {
        const double lo = fmin(x, y), hi = fmax(x, y);
        x = lo;
        y = hi;
    };
    cx(a[0], a[1]); cx(a[2], a[3]); cx(a[4], a[5]); cx(a[6], a[7]);
    cx(a[0], a[2]); cx(a[1], a[3]); cx(a[4], a[6]); cx(a[5], a[7]);
    cx(a[1], a[2]); cx(a[5], a[6]); cx(a[0], a[4]); cx(a[3], a[7]);
    cx(a[1], a[5]); cx(a[2], a[6]);
    cx(a[1], a[4]); cx(a[3], a[6]);
    cx(a[2], a[4]); cx(a[3], a[5]);
    cx(a[3], a[4]);
}

// Mean and both percentile lists of the samples' times.  Whole groups of eight samples are sorted once (shared by the list of
// the smallest and the list of the largest) and merged into the lists: 12.5 instead of 28 minimum / maximum operations
// per sample.
struct SweepStat {
    ExtremeK<false> lo;
    ExtremeK<true> hi;
    double sum;
    __device__ void init() {
        lo.init();
        hi.init();
        sum = 0.0;
    }
    __device__ void take(double (&a)[kSweepGroup]) {
        sum += ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
        sort_group(a);
        lo.merge(a);
        hi.merge(a);
    }
    __device__ void take_one(double a) {
        sum += a;
        lo.push(a);
        hi.push(a);
    }
};

// One setting of the seven slower axes.
struct ExpandTile {
    uint32_t row;                               // (model, tp, precision) row of coefficients
    uint32_t model, hw, b, d_sin, s_in, s_out, d_tp, p, wbits;
};
__device__ inline ExpandTile expand_tile(const GridLds &s, const GridDesc &g, uint32_t tile) {
    uint32_t dg[AX_BLK], rem = tile;
#pragma unroll
    for (int a = AX_BLK - 1; a > 0; --a) {
        const uint32_t q = div32(rem, g.div[a]);
        dg[a] = rem - q * g.div[a].d;
        rem = q;
    }
    dg[0] = rem;
    ExpandTile t;
    t.row = (dg[AX_MODEL] * g.div[AX_TP].d + dg[AX_TP]) * g.div[AX_WBITS].d + dg[AX_WBITS];
    t.model = s.axis[AX_MODEL][dg[AX_MODEL]];
    t.hw = s.axis[AX_HW][dg[AX_HW]];
    t.b = s.axis[AX_BATCH][dg[AX_BATCH]];
    t.d_sin = dg[AX_SIN];
    t.s_in = s.axis[AX_SIN][dg[AX_SIN]];
    t.s_out = s.axis[AX_SOUT][dg[AX_SOUT]];
    t.d_tp = dg[AX_TP];
    t.p = s.axis[AX_TP][dg[AX_TP]];
    t.wbits = s.axis[AX_WBITS][dg[AX_WBITS]];
    return t;
}

// Efficiency sweep.  Neither latency depends on the KV block size, so one lane evaluates the samples
// for all block sizes of a configuration at once (rows that differ only in the kv_block digit) and
// only the memory check is repeated per block size.
//
// A sample scales every compute time by x = 1 / e_c and every read time by y = 1 / e_b.  A configuration's time is a sum of
// terms max(F x, B y) -- one per task and pass, with the passes' counts multiplied in -- plus the transfers.  F and B are
// added up as operations and bytes, whose sums are whole numbers or nearly so, and turned into times last: the roundings
// of a configuration's sums are common to all its samples and do not average out in the means.  Over the
// ratios x / y of all samples most terms are bound by the same side throughout: those are added up once per
// configuration, and a sample costs two multiply-adds for all of them.  The others (a few per wave: neighbouring
// configurations have them in common) are kept as pairs and evaluated per sample, skipped by branches that are uniform
// over the wave.
//
// A configuration's outputs are the same bits whichever variant of the kernel a range is given to, so sums are contracted where
// the code says fma and nowhere else (here and in what it calls: make_coef, attention_series).  A term of a neighbour in
// the wave adds zero.

// Work items of a sweep.  The first n_prefill (a multiple of a wave, or none) are settings of all axes but s_out and kv_block, of which
// only the prefill's columns are made, n_s_out * NB rows at a time; the others are settings of all axes but kv_block.
struct SweepItems {
    uint32_t n, n_prefill;          // items; those of the prefill
    uint32_t prefill_end;           // the last ones up to n_prefill are empty
    uint32_t first_group, inner;    // the first setting of the axes above s_out that holds rows of the range; tiles from a value of s_out to the next
};

constexpr double kLargest = 0x1.fffffffffffffp+1023;
constexpr int kPassTerms = N_LINEAR + 2;                // the linear tasks, attention, LM head
template <int N>
struct SweepTerms {
    double F[N], B[N];          // terms that change sides within the samples (0, 0 in lanes where they do not)
    double a_F, a_B, fixed;     // the other terms' sums; transfers
    uint32_t active;            // wave-uniform: terms that change sides in some lane
    __device__ void init() {
        a_F = a_B = fixed = 0.0;
        active = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) F[i] = B[i] = 0.0;
    }
    // a term of n x per operations and b bytes
    template <bool ADDITIVE>
    __device__ void add(int i, double n, double per, double b, double rho_lo, double rho_hi) {
#pragma clang fp contract(off)
        const double f = n * per;
        const bool compute = ADDITIVE || f * rho_lo >= b, read = ADDITIVE || f * rho_hi <= b;
        a_F = ADDITIVE ? fma(n, per, a_F) : a_F + (compute ? f : 0.0);
        a_B += read && (ADDITIVE || !compute) ? b : 0.0;
        if (!ADDITIVE) {
            const bool both = !compute && !read;
            F[i] = both ? f : 0.0;
            B[i] = both ? b : 0.0;
        }
    }
    // `times` passes of T tokens with attention workload Q, K context tokens and n_lm LM-head rows; att: attention counts
    template <bool ADDITIVE>
    __device__ void add_pass(int i0, const Coef &c, const HwRecip &hw, double times, double T, double Q, double K, double n_lm,
                             bool att, double rho_lo, double rho_hi) {
#pragma clang fp contract(off)
        const double w = times * c.L, wT = w * T, w_eld = w * fmin(c.E, c.k * T), lm = times * n_lm;
#pragma unroll
        for (int i = 0; i < N_LINEAR; ++i) {
            const bool experts = i == OP_UP || i == OP_DOWN;
            add<ADDITIVE>(i0 + i, wT, c.f[i], fma(wT, c.a[i], (experts ? w_eld : w) * c.w[i]), rho_lo, rho_hi);
        }
        if (att) add<ADDITIVE>(i0 + N_LINEAR, w * Q, c.f_att, fma(w * K, c.c_att, wT * c.a_att), rho_lo, rho_hi);
        if (n_lm > 0.0) add<ADDITIVE>(i0 + N_LINEAR + 1, lm, c.f_lm, fma(lm, c.a_lm, times * c.w_lm), rho_lo, rho_hi);
        a_B = fma(wT, c.a_nm, a_B);
        fixed = fma(2.0, fma(wT * c.m_ar, hw.r_link, w * c.n_ar * hw.lat), fixed);
    }
    // operations and bytes become seconds; to be called by all lanes in action together, after the last add
    __device__ void settle(const HwRecip &hw) {
        a_F *= hw.r_peak;
        a_B *= hw.r_bw;
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (__ballot(F[i] != 0.0)) {                // (a term that changes sides has F > 0)
                m |= 1u << i;
                F[i] *= hw.r_peak;
                B[i] *= hw.r_bw;
            }
        }
        active = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
    }
    template <int G>
    __device__ void evaluate(const double (&x)[G], const double (&y)[G], double (&v)[G]) const {
#pragma unroll
        for (int q = 0; q < G; ++q) v[q] = fma(x[q], a_F, fma(y[q], a_B, fixed));
#pragma unroll
        for (int i0 = 0; i0 < N; i0 += kPassTerms) {
            if (((active >> i0) & ((1u << kPassTerms) - 1u)) == 0u) continue;       // no term of the pass
#pragma unroll
            for (int i = i0; i < i0 + kPassTerms; ++i) {
                if ((active >> i) & 1u) {
#pragma unroll
                    for (int q = 0; q < G; ++q) v[q] = fmax(fma(F[i], x[q], v[q]), fma(B[i], y[q], v[q]));
                }
            }
        }
    }
};

// SHARED: the prefill's columns, which are the same for all values of s_out, are made by items of their own; the others then sort
// one metric instead of two.  (One lane for several values of s_out, with the prefill's columns once for all of them, is slower,
// 145 - 170 us: the waves whose terms change sides take three times as long as the others, and fewer, longer items do not even that out.)
// Bound by the vector ALU, two waves per SIMD.  1.9 million configurations x 64 samples: 115 - 124 us a call by inputs and device, of which the
// set-up and the stores are about 55 (a call with three samples takes 60); 142 with one item for all columns as well (8 more with products and sums of a
// term that changes sides apart and the samples added one by one); 405 us with every task's two sides, the split of the series and the coefficients
// worked out per sample.  The samples' factors in scalar registers instead of vector registers: 10 % slower.  Samples in the order of
// their ratios, so that a term changes sides in few groups of eight and is added up once per group elsewhere, gain nothing: finding
// the groups costs what it saves.
template <bool ADDITIVE, bool SHARED>
__global__ __launch_bounds__(kBlock, 2) void eval_sweep_kernel(GridDesc g, const DevTables *__restrict__ tab,
                                                            uint32_t first, uint32_t count, uint32_t n_eff,
                                                            guide_stats out, const TileLds *__restrict__ derived,
                                                            SweepItems items) {
#pragma clang fp contract(off)
    __shared__ TileLds s;
    __shared__ double2 s_eff[GUIDE_MAX_EFF];            // (1 / e_c, 1 / e_b)
    __shared__ double s_rho[GUIDE_MAX_EFF], s_balance[GUIDE_MAX_HW];
    const uint32_t n_rows = g.div[AX_MODEL].d * g.div[AX_TP].d * g.div[AX_WBITS].d;
    const bool coef_in_lds = n_rows <= kCoefRows;
    {
        const uint32_t vecs = (uint32_t)(offsetof(TileLds, coef) + (coef_in_lds ? n_rows : 0u) * sizeof(Coef) + 15) / 16;
        for (uint32_t i = threadIdx.x; i < vecs; i += kBlock) ((uint4 *)&s)[i] = ((const uint4 *)derived)[i];
    }
    for (uint32_t i = threadIdx.x; i < g.n_hw; i += blockDim.x) {
        const HwRecip &hw = derived->g.hw[i];
        s_balance[i] = hw.r_peak / hw.r_bw;
    }
    for (uint32_t i = threadIdx.x; i < n_eff; i += blockDim.x) {
        // (finite also for subnormal efficiencies: a sum of no terms times infinity would be no number, and would
        // drop out of the sorting instead of coming last)
        s_eff[i] = double2{fmin(1.0 / tab->eff_c[i], kLargest), fmin(1.0 / tab->eff_b[i], kLargest)};
        s_rho[i] = fmin(tab->eff_b[i] / tab->eff_c[i], kLargest);
    }
    __syncthreads();
    double rho_lo = s_rho[0], rho_hi = rho_lo;                      // least and largest x / y
    for (uint32_t e = 1; e < n_eff; ++e) {
        rho_lo = fmin(rho_lo, s_rho[e]);
        rho_hi = fmax(rho_hi, s_rho[e]);
    }
    // (a rounding of rho decides a term only where both sides are equal to rounding)
    // nearest rank: p10 = sorted[ceil(n/10) - 1]; p90 = sorted[ceil(9n/10) - 1] = (n - ceil(9n/10))-th largest, 0-based
    const uint32_t r_lo = (n_eff + 9) / 10 - 1;
    const uint32_t r_hi = n_eff - (9 * n_eff + 9) / 10;
    const uint32_t NB = g.div[AX_BLK].d, NM = g.div[AX_MBT].d, TS = NB * NM;
    const uint32_t last = first + count, n_s_out = g.div[AX_SOUT].d, t_first = first / TS;
    for (uint32_t u = blockIdx.x * kBlock + threadIdx.x; u < items.n; u = stride_on(u, gridDim.x * kBlock, items.n)) {
        const bool prefill_only = SHARED && u < items.n_prefill;                    // (the same in a whole wave)
        const uint32_t w = SHARED && !prefill_only ? u - items.n_prefill : u;
        const uint32_t q = w / NM, m_digit = w - q * NM;
        uint32_t hi = t_first + q, steps = 1;                     // tile; values of s_out
        if (prefill_only) {
            const uint32_t group = q / items.inner;
            hi = (items.first_group + group) * (n_s_out * items.inner) + (q - group * items.inner);
            steps = n_s_out;
        }
        uint32_t row0 = hi * TS + m_digit;                        // the row with kv_block digit 0
        // none of this item's rows inside [first, last)?  (only at the ragged ends)
        if ((prefill_only && u >= items.prefill_end) || row0 + ((steps - 1) * items.inner * NB + NB - 1) * NM < first || row0 >= last) continue;
        const ExpandTile tl = expand_tile(s.g, g, hi);
        const uint32_t mbt = s.g.axis[AX_MBT][m_digit];
        const HwRecip hw = s.g.hw[tl.hw];
        const Coef cf = coef_in_lds ? s.coef[tl.row] : make_coef(s.g.models[tl.model], tl.p, tl.wbits, s.r_tp[tl.d_tp]);
        // the ratios in operations and bytes (finite: no operations times infinity would be no number)
        const double lo = fmin(rho_lo * s_balance[tl.hw], kLargest), up = fmin(rho_hi * s_balance[tl.hw], kLargest);
        const PrefillPlan plan = make_prefill_plan(tl.b, tl.s_in, mbt, s.r_sin[tl.d_sin], s.r_mbt[m_digit]);
        SweepTerms<2 * kPassTerms> pre;
        SweepTerms<kPassTerms> dec;
        pre.init();
        // attention over the full segments of a long prompt, or over the decode steps, is a series of terms; where it
        // changes sides within the samples it is summed per sample
        double p_al = 0.0, p_be = 0.0, p_ga = 0.0, d_al = 0.0, d_be = 0.0, d_ga = 0.0;
        bool p_series = false, d_series = false;
        const double b = (double)tl.b, S = plan.S;
        double n = 0.0;                                           // decode steps
        // sum over contexts first, 2 first, .. or s + 1, .., s + n: both sides are linear in the context, so the ends decide.
        // n_al, n_be, n_ga: whole numbers that multiply the operations per pair, the cache and the activation bytes.
        auto series = [&](auto &terms, double n_al, double n_be, double n_ga, double c_lo, double c_hi, double all,
                          double steps, double &o_al, double &o_be, double &o_ga) {
            const double al = n_al * cf.f_att, be = n_be * cf.c_att, ga = n_ga * cf.a_att;
            const bool read = ADDITIVE || al * up * c_hi <= fma(be, c_hi, ga);
            const bool compute = ADDITIVE || al * lo * c_lo >= fma(be, c_lo, ga);
            terms.a_F = ADDITIVE ? fma(n_al * all, cf.f_att, terms.a_F) : terms.a_F + (compute ? (n_al * all) * cf.f_att : 0.0);
            terms.a_B += read && (ADDITIVE || !compute) ? fma(n_be * all, cf.c_att, (n_ga * steps) * cf.a_att) : 0.0;
            const bool both = !read && !compute;
            o_al = both ? al * hw.r_peak : 0.0;
            o_be = both ? be * hw.r_bw : 0.0;
            o_ga = both ? ga * hw.r_bw : 0.0;
            return both;
        };
        const bool seg = plan.segmented;
        const double R = plan.R, bL = b * cf.L;
        pre.add_pass<ADDITIVE>(0, cf, hw, seg ? b * plan.n_fs : plan.n_full, seg ? plan.M : R * S, R * S * S, R * S, R, !seg,
                               lo, up);
        if (seg || plan.rem > 0.0)
            pre.add_pass<ADDITIVE>(kPassTerms, cf, hw, seg ? b : 1.0, seg ? plan.c_last : plan.rem * S,
                                   seg ? plan.c_last * S : plan.rem * S * S, seg ? S : plan.rem * S, seg ? 1.0 : plan.rem, true,
                                   lo, up);
        if (seg)
            p_series = series(pre, bL * plan.M, bL, bL * plan.M, plan.M, plan.n_fs * plan.M,
                              plan.M * (0.5 * plan.n_fs * (plan.n_fs + 1.0)), plan.n_fs, p_al, p_be, p_ga);
        pre.settle(hw);
        const bool any_p = __ballot(p_series) != 0;             // wave-uniform
        dec.init();
        if (!prefill_only && tl.s_out > 1) {
            n = (double)(tl.s_out - 1);
            dec.add_pass<ADDITIVE>(0, cf, hw, n, b, 0.0, 0.0, b, false, lo, up);
            d_series = series(dec, bL, bL, bL, S + 1.0, S + n, fma(n, S, 0.5 * n * (n + 1.0)), n, d_al, d_be, d_ga);
        }
        dec.settle(hw);
        const bool any_d = __ballot(d_series) != 0;
        auto efficiencies = [&](uint32_t e, auto &x, auto &y) {
            constexpr int G = sizeof(x) / sizeof(double);
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const double2 ef = s_eff[e + q];        // (moved to scalar registers, four instructions a sample: 10 % slower)
                x[q] = ef.x;
                y[q] = ef.y;
            }
        };
        auto prefill_times = [&](const auto &x, const auto &y, auto &tp) {
            constexpr int G = sizeof(tp) / sizeof(double);
            pre.evaluate(x, y, tp);
            if (any_p) {
#pragma unroll
                for (int q = 0; q < G; ++q)
                    tp[q] += attention_series<ADDITIVE>(p_al * x[q], p_be * y[q], p_ga * y[q], 0.0, plan.M, plan.r_mbt, plan.n_fs);
            }
        };
        auto batch_times = [&](const auto &x, const auto &y, const auto &tp, auto &tb) {
            constexpr int G = sizeof(tb) / sizeof(double);
            if (prefill_only) {
#pragma unroll
                for (int q = 0; q < G; ++q) tb[q] = tp[q];
                return;
            }
            dec.evaluate(x, y, tb);
            if (any_d) {
#pragma unroll
                for (int q = 0; q < G; ++q)
                    tb[q] += attention_series<ADDITIVE>(d_al * x[q], d_be * y[q], d_ga * y[q], S, 1.0, 1.0, n);
            }
#pragma unroll
            for (int q = 0; q < G; ++q) tb[q] += tp[q];
        };
        SweepStat st_p, st_b;                                     // SHARED: st_b alone, of the prefill or of the batch
        st_p.init();
        st_b.init();
        uint32_t e = 0;
        for (; e + kSweepGroup <= n_eff; e += kSweepGroup) {
            double x[kSweepGroup], y[kSweepGroup], tp[kSweepGroup], tb[kSweepGroup];
            efficiencies(e, x, y);
            prefill_times(x, y, tp);
            batch_times(x, y, tp, tb);
            if (!SHARED) st_p.take(tp);
            st_b.take(tb);
        }
        for (; e < n_eff; ++e) {
            double x[1], y[1], tp[1], tb[1];
            efficiencies(e, x, y);
            prefill_times(x, y, tp);
            batch_times(x, y, tp, tb);
            if (!SHARED) st_p.take_one(tp[0]);
            st_b.take_one(tb[0]);
        }
        const double mean_b = st_b.sum / (double)n_eff, p10_b = st_b.lo.at(r_lo), p90_b = st_b.hi.at(r_hi);
        auto put_prefill = [&](uint32_t i, double mean, double p10, double p90) {
            if (out.ttft_mean) out.ttft_mean[i] = mean;
            if (out.ttft_p10) out.ttft_p10[i] = p10;
            if (out.ttft_p90) out.ttft_p90[i] = p90;
        };
        if (prefill_only) {
            for (uint32_t step = 0; step < steps; ++step, row0 += items.inner * TS) {
                for (uint32_t k = 0; k < NB; ++k) {
                    const uint32_t row = row0 + k * NM;
                    if (row >= first && row < last) put_prefill(row - first, mean_b, p10_b, p90_b);
                }
            }
            continue;
        }
        double mean_p = 0.0, p10_p = 0.0, p90_p = 0.0;
        if (!SHARED) {
            mean_p = st_p.sum / (double)n_eff;
            p10_p = st_p.lo.at(r_lo);
            p90_p = st_p.hi.at(r_hi);
        }
        const double cost = (double)tl.p * mean_b / 3600.0 * 1.0e6 / (b * (double)tl.s_out);
        for (uint32_t k = 0; k < NB; ++k) {
            const uint32_t row = row0 + k * NM;
            if (row < first || row >= last) continue;
            const uint32_t i = row - first;
            if (!SHARED) put_prefill(i, mean_p, p10_p, p90_p);
            if (out.t_batch_mean) out.t_batch_mean[i] = mean_b;
            if (out.t_batch_p10) out.t_batch_p10[i] = p10_b;
            if (out.t_batch_p90) out.t_batch_p90[i] = p90_b;
            if (out.cost) out.cost[i] = cost;
            if (out.b_max || out.feasible) {
                const MemResult mem = memory_check(cf.w_gpu, cf.kv_tok, hw.cap, tl.b, tl.s_in, tl.s_out, s.g.axis[AX_BLK][k]);
                if (out.b_max) out.b_max[i] = mem.b_max;
                if (out.feasible) out.feasible[i] = mem.feasible ? 1 : 0;
            }
        }
    }
}

// ---------------------------------------------------------------- expanded variants
//
// Where a lane cannot own a whole tile (more than four values on one of the two fastest axes) or hardly any column varies
// inside one (the cluster-level columns), a block takes a run of tiles, works out into LDS what depends on the tile,
// on (tile, token budget) and on (tile, block size), and then writes the rows from there, each wave 64 consecutive
// rows of every column.

constexpr uint32_t kExpandTiles = 256;          // most tiles of a run
constexpr uint32_t kExpandParts = 1024;         // most (tile, block size) and (tile, token budget) pairs of a run
template <bool STREAM, typename T>
__device__ inline void put(T *col, uint32_t i, T v) {
    if (STREAM) __builtin_nontemporal_store(v, &col[i]);
    else col[i] = v;
}

// What the two kernels below share, so that a row's values are the same bits in either.
__device__ inline double tile_tok_s(const ExpandTile &tl, double t_dec) {
    return tl.s_out > 1 ? (double)tl.b * (double)(tl.s_out - 1) / t_dec : 0.0;
}
// Cost per second of the batch.  (Divisions here and above: their operands are exact, t_dec apart, so both columns have
// two roundings at most.)
__device__ inline double tile_cost(const ExpandTile &tl) {
    return (double)tl.p * 1.0e6 / (3600.0 * ((double)tl.b * (double)tl.s_out));
}
__device__ inline MemResult tile_memory(const Coef &cf, double cap, const ExpandTile &tl, uint32_t blk, double r_blk) {
    MemResult m;
    const double c_avail = cap - cf.w_gpu;
    const uint32_t tok_req = floor_div(tl.s_in + tl.s_out + blk - 1, r_blk) * blk;
    const double kv_req = (double)tok_req * cf.kv_tok;
    const double q = floor(c_avail / kv_req);
    const bool room = c_avail > 0.0;
    m.b_max = !room ? 0u : (q >= 4294967295.0 ? 4294967295u : (uint32_t)q);
    m.feasible = room && (double)tl.b * kv_req <= c_avail;
    return m;
}
// What a block needs of the derived tables; the coefficients when they fit.
__device__ inline bool stage_tile_tables(TileLds &s, const GridDesc &g, const TileLds *__restrict__ derived) {
    const uint32_t n_rows = g.div[AX_MODEL].d * g.div[AX_TP].d * g.div[AX_WBITS].d;
    const bool coef_in_lds = n_rows <= kCoefRows;
    const uint32_t vecs = (uint32_t)(offsetof(TileLds, coef) + (coef_in_lds ? n_rows : 0u) * sizeof(Coef) + 15) / 16;
    for (uint32_t i = threadIdx.x; i < vecs; i += kBlock) ((uint4 *)&s)[i] = ((const uint4 *)derived)[i];
    return coef_in_lds;
}

// Evaluation of grids with more than four values on one of the two fastest axes.  per_run: tiles of a run.
// Bound by latency and launch at ordinary sizes: 443 211 rows of a grid with five block sizes and six token
// budgets (20 MB), additive times: 8.6 us (124 vector instructions per row); one index per lane, which repeats the decode
// series and the prefill for every row: 22.9 us.
template <bool ADDITIVE, bool STREAM>
__global__ __launch_bounds__(kBlock) void eval_wide_kernel(GridDesc g, uint32_t first, uint32_t count, double re_c,
                                                           double re_b, guide_metrics out,
                                                           const TileLds *__restrict__ derived, uint32_t per_run) {
    __shared__ TileLds s;
    __shared__ ExpandTile s_tile[kExpandTiles];
    __shared__ double s_dec[kExpandTiles], s_tok[kExpandTiles], s_cost[kExpandTiles], s_pre[kExpandParts];
    __shared__ uint32_t s_bmax[kExpandParts];
    __shared__ uint8_t s_feas[kExpandParts];
    const bool coef_in_lds = stage_tile_tables(s, g, derived);
    __syncthreads();
    const uint32_t NB = g.div[AX_BLK].d, NM = g.div[AX_MBT].d, TS = NB * NM;
    const uint32_t t_first = first / TS, last = first + count, n_tiles = (last - 1) / TS - t_first + 1;
    for (uint64_t run64 = (uint64_t)blockIdx.x * per_run; run64 < n_tiles; run64 += (uint64_t)gridDim.x * per_run) {
        const uint32_t run = (uint32_t)run64, tiles = n_tiles - run < per_run ? n_tiles - run : per_run;
        for (uint32_t t = threadIdx.x; t < tiles; t += kBlock) s_tile[t] = expand_tile(s.g, g, t_first + run + t);
        __syncthreads();
        // items: a decode series per tile, a prefill per (tile, token budget), a memory check per (tile, block size)
        const uint32_t n_pre = tiles * NM, n_mem = tiles * NB, n_items = tiles + n_pre + n_mem;
        for (uint32_t i = threadIdx.x; i < n_items; i += kBlock) {
            uint32_t t, part = 0;
            if (i < n_pre) {
                t = div32(i, g.div[AX_MBT]);
                part = i - t * NM;
            } else if (i < n_pre + tiles) {
                t = i - n_pre;
            } else {
                t = div32(i - n_pre - tiles, g.div[AX_BLK]);
                part = i - n_pre - tiles - t * NB;
            }
            const ExpandTile tl = s_tile[t];
            const Coef cf = coef_in_lds ? s.coef[tl.row] : make_coef(s.g.models[tl.model], tl.p, tl.wbits, s.r_tp[tl.d_tp]);
            const HwRecip hw = s.g.hw[tl.hw];
            if (i < n_pre + tiles) {
                const TimeCoef tc = make_time_coef(cf, hw.r_peak * re_c, hw.r_bw * re_b, hw.r_link, hw.lat);
                if (i < n_pre) {
                    s_pre[i] = prefill_time_fast<ADDITIVE>(tc, tl.b, tl.s_in, s.g.axis[AX_MBT][part], s.r_sin[tl.d_sin],
                                                           s.r_mbt[part]);
                } else {
                    const double t_dec = decode_time_fast<ADDITIVE>(tc, tl.b, tl.s_in, tl.s_out - 1);
                    s_dec[t] = t_dec;
                    s_tok[t] = tile_tok_s(tl, t_dec);
                    s_cost[t] = tile_cost(tl);
                }
            } else {
                const MemResult m = tile_memory(cf, hw.cap, tl, s.g.axis[AX_BLK][part], s.r_blk[part]);
                s_bmax[t * NB + part] = m.b_max;
                s_feas[t * NB + part] = m.feasible ? 1 : 0;
            }
        }
        __syncthreads();
        const uint32_t row0 = (t_first + run) * TS;             // grid index of the run's first row
        const uint32_t lo = row0 > first ? row0 : first;
        const uint32_t skip = lo - row0, in_run = tiles * TS - skip, n = last - lo < in_run ? last - lo : in_run;
        for (uint32_t j = blockIdx.y * kBlock + threadIdx.x; j < n; j += gridDim.y * kBlock) {
            const uint32_t rel = skip + j, tk = div32(rel, g.div[AX_MBT]), m = rel - tk * NM, t = div32(tk, g.div[AX_BLK]);
            const uint32_t i = lo - first + j;
            const double t_pre = s_pre[t * NM + m], t_dec = s_dec[t], t_batch = t_pre + t_dec;
            if (out.t_prefill) put<STREAM>(out.t_prefill, i, t_pre);
            if (out.t_decode) put<STREAM>(out.t_decode, i, t_dec);
            if (out.t_batch) put<STREAM>(out.t_batch, i, t_batch);
            if (out.decode_tok_s) put<STREAM>(out.decode_tok_s, i, s_tok[t]);
            if (out.cost) put<STREAM>(out.cost, i, t_batch * s_cost[t]);
            if (out.b_max) out.b_max[i] = s_bmax[tk];
            if (out.feasible) out.feasible[i] = s_feas[tk];
        }
        __syncthreads();                                        // the run's values have been read
    }
}

// The same for few rows, one index per lane: no phases to wait for.
template <bool ADDITIVE>
__global__ __launch_bounds__(kBlock) void eval_wide_rows_kernel(GridDesc g, uint32_t first, uint32_t count, double re_c,
                                                                double re_b, guide_metrics out,
                                                                const TileLds *__restrict__ derived) {
    __shared__ TileLds s;
    const bool coef_in_lds = stage_tile_tables(s, g, derived);
    __syncthreads();
    const uint32_t NB = g.div[AX_BLK].d, NM = g.div[AX_MBT].d;
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < count; i = stride_on(i, gridDim.x * kBlock, count)) {
        const uint32_t tk = div32(first + i, g.div[AX_MBT]), m = first + i - tk * NM, t = div32(tk, g.div[AX_BLK]), k = tk - t * NB;
        const ExpandTile tl = expand_tile(s.g, g, t);
        const Coef cf = coef_in_lds ? s.coef[tl.row] : make_coef(s.g.models[tl.model], tl.p, tl.wbits, s.r_tp[tl.d_tp]);
        const HwRecip hw = s.g.hw[tl.hw];
        const TimeCoef tc = make_time_coef(cf, hw.r_peak * re_c, hw.r_bw * re_b, hw.r_link, hw.lat);
        const double t_pre = prefill_time_fast<ADDITIVE>(tc, tl.b, tl.s_in, s.g.axis[AX_MBT][m], s.r_sin[tl.d_sin], s.r_mbt[m]);
        const double t_dec = decode_time_fast<ADDITIVE>(tc, tl.b, tl.s_in, tl.s_out - 1);
        double t_batch;
        {
#pragma clang fp contract(off)                                  // a sum of two rounded values, as in the other kernel
            t_batch = t_pre + t_dec;
        }
        const MemResult mem = tile_memory(cf, hw.cap, tl, s.g.axis[AX_BLK][k], s.r_blk[k]);
        if (out.t_prefill) out.t_prefill[i] = t_pre;
        if (out.t_decode) out.t_decode[i] = t_dec;
        if (out.t_batch) out.t_batch[i] = t_batch;
        if (out.decode_tok_s) out.decode_tok_s[i] = tile_tok_s(tl, t_dec);
        if (out.cost) out.cost[i] = t_batch * tile_cost(tl);
        if (out.b_max) out.b_max[i] = mem.b_max;
        if (out.feasible) out.feasible[i] = mem.feasible ? 1 : 0;
    }
}

// Cluster-level columns under a GPU budget: every one depends on the tile, on (tile, block size) or on (tile, token
// budget) alone, so the rows are copies.  Bound by the stores: the full grid's twelve columns (57 bytes a row, 108 MB)
// take 26 us (227 vector instructions per row); one index per lane with everything worked out per row (571) took 49 us.
template <bool ADDITIVE, bool STREAM>
__global__ __launch_bounds__(kBlock) void eval_extras_kernel(GridDesc g, const DevTables *__restrict__ tab,
                                                             uint32_t first, uint32_t count, uint32_t n_gpus,
                                                             guide_extras out, uint32_t per_run) {
    __shared__ GridLds s;
    __shared__ ExpandTile s_tile[kExpandTiles];
    __shared__ double s_avail[kExpandTiles], s_kv[kExpandTiles], s_cluster[kExpandTiles], s_paper[kExpandTiles];
    __shared__ uint32_t s_smax[kExpandTiles], s_dp[kExpandTiles], s_sadj[kExpandTiles], s_skept[kExpandTiles];
    __shared__ uint64_t s_par[kExpandParts];
    __shared__ uint32_t s_badj[kExpandParts], s_bkept[kExpandParts], s_sub[kExpandParts], s_seg[kExpandParts];
    __shared__ uint8_t s_fkept[kExpandParts];
    stage_grid_tables(s, g, tab);
    __syncthreads();
    const uint32_t NB = g.div[AX_BLK].d, NM = g.div[AX_MBT].d, TS = NB * NM;
    const uint32_t t_first = first / TS, last = first + count, n_tiles = (last - 1) / TS - t_first + 1;
    const double keep = out.kv_keep == 0.0 ? 1.0 : out.kv_keep;
    const bool any_tok = out.cluster_tok_s || out.paper_tok_s, any_kept = out.b_max_kept || out.feasible_kept;
    for (uint64_t run64 = (uint64_t)blockIdx.x * per_run; run64 < n_tiles; run64 += (uint64_t)gridDim.x * per_run) {
        const uint32_t run = (uint32_t)run64, tiles = n_tiles - run < per_run ? n_tiles - run : per_run;
        for (uint32_t t = threadIdx.x; t < tiles; t += kBlock) {
            const ExpandTile tl = expand_tile(s, g, t_first + run + t);
            const HwRecip hw = s.hw[tl.hw];
            const Coef cf = make_coef(s.models[tl.model], tl.p, tl.wbits);
            const uint32_t dp = n_gpus / tl.p;
            double tok_s = 0.0, tok_s1 = 0.0;
            if (tl.s_out > 1 && any_tok) {
                const double n = (double)tl.b * (double)(tl.s_out - 1);
                const TimeCoef tc = make_time_coef(cf, hw.r_peak, hw.r_bw, hw.r_link, hw.lat);
                tok_s = n / decode_time<ADDITIVE>(tc, tl.b, tl.s_in, tl.s_out - 1);
                if (out.paper_tok_s) {
                    const Coef c1 = make_coef(s.models[tl.model], 1u, tl.wbits);   // the same candidate on one GPU
                    const TimeCoef t1 = make_time_coef(c1, hw.r_peak, hw.r_bw, hw.r_link, hw.lat);
                    tok_s1 = n / decode_time<ADDITIVE>(t1, tl.b, tl.s_in, tl.s_out - 1);
                }
            }
            const double c_avail = hw.cap - cf.w_gpu;
            const bool room = c_avail > 0.0;
            const double q = floor(c_avail / ((double)tl.b * cf.kv_tok)), qs = floor(q / keep);
            const uint32_t s_max = !room ? 0u : (q >= 4294967295.0 ? 4294967295u : (uint32_t)q);
            const uint32_t len = tl.s_in + tl.s_out;                    // both below 2^31
            s_tile[t] = tl;
            s_avail[t] = c_avail;
            s_kv[t] = cf.kv_tok;
            s_cluster[t] = (double)dp * tok_s;
            s_paper[t] = ((double)dp * (double)tl.p) * tok_s1 / (1.0 + log2((double)tl.p));
            s_smax[t] = s_max;
            s_dp[t] = dp;
            s_sadj[t] = len < s_max ? len : s_max;
            s_skept[t] = !room ? 0u : (qs >= 4294967295.0 ? 4294967295u : (uint32_t)qs);
        }
        __syncthreads();
        const uint32_t n_mem = tiles * NB, n_pre = tiles * NM;
        for (uint32_t i = threadIdx.x; i < n_mem + n_pre; i += kBlock) {
            if (i < n_mem) {
                const uint32_t t = div32(i, g.div[AX_BLK]), blk = s.axis[AX_BLK][i - t * NB];
                const ExpandTile tl = s_tile[t];
                const double c_avail = s_avail[t];
                const bool room = c_avail > 0.0;
                const uint32_t len = tl.s_in + tl.s_out;
                const uint32_t tok_req = (len + blk - 1) / blk * blk;
                const double qb = floor(c_avail / ((double)tok_req * s_kv[t]));
                const uint32_t b_max = !room ? 0u : (qb >= 4294967295.0 ? 4294967295u : (uint32_t)qb);
                s_par[i] = (uint64_t)s_dp[t] * (uint64_t)b_max;
                s_badj[i] = tl.b < b_max ? tl.b : b_max;
                if (any_kept) {
                    // a KV-cache reduction that keeps the fraction kv_keep of every request's entries
                    const uint64_t kept = (uint64_t)ceil(keep * (double)len);
                    const double kv_req = (double)((kept + blk - 1) / blk * blk) * s_kv[t];
                    const double qk = floor(c_avail / kv_req);
                    s_bkept[i] = !room ? 0u : (qk >= 4294967295.0 ? 4294967295u : (uint32_t)qk);
                    s_fkept[i] = (room && (double)tl.b * kv_req <= c_avail) ? 1 : 0;
                }
            } else {
                const uint32_t j = i - n_mem, t = div32(j, g.div[AX_MBT]), mbt = s.axis[AX_MBT][j - t * NM];
                const uint32_t b = s_tile[t].b, s_in = s_tile[t].s_in;
                const bool long_prompt = s_in > mbt;
                uint32_t split = mbt / s_in;                            // prompts per pass (0 for a long prompt)
                split = split < b ? split : b;
                s_sub[j] = long_prompt ? b : (b + split - 1) / split;
                s_seg[j] = long_prompt ? (s_in - 1) / mbt + 1 : 1u;
            }
        }
        __syncthreads();
        const uint32_t row0 = (t_first + run) * TS;
        const uint32_t lo = row0 > first ? row0 : first;
        const uint32_t skip = lo - row0, in_run = tiles * TS - skip, n = last - lo < in_run ? last - lo : in_run;
        for (uint32_t j = blockIdx.y * kBlock + threadIdx.x; j < n; j += gridDim.y * kBlock) {
            const uint32_t rel = skip + j, tk = div32(rel, g.div[AX_MBT]), m = rel - tk * NM, t = div32(tk, g.div[AX_BLK]);
            const uint32_t i = lo - first + j, tm = t * NM + m;
            if (out.s_max) put<STREAM>(out.s_max, i, s_smax[t]);
            if (out.dp_max) put<STREAM>(out.dp_max, i, s_dp[t]);
            if (out.max_parallelism) put<STREAM>(out.max_parallelism, i, s_par[tk]);
            if (out.cluster_tok_s) put<STREAM>(out.cluster_tok_s, i, s_cluster[t]);
            if (out.paper_tok_s) put<STREAM>(out.paper_tok_s, i, s_paper[t]);
            if (out.b_adj) put<STREAM>(out.b_adj, i, s_badj[tk]);
            if (out.n_sub_batches) put<STREAM>(out.n_sub_batches, i, s_sub[tm]);
            if (out.n_segments) put<STREAM>(out.n_segments, i, s_seg[tm]);
            if (out.s_adj) put<STREAM>(out.s_adj, i, s_sadj[t]);
            if (out.b_max_kept) put<STREAM>(out.b_max_kept, i, s_bkept[tk]);
            if (out.s_max_kept) put<STREAM>(out.s_max_kept, i, s_skept[t]);
            if (out.feasible_kept) out.feasible_kept[i] = s_fkept[tk];
        }
        __syncthreads();                                        // the run's values have been read
    }
}

// Cluster-level columns for few rows, one index per lane: no phases to wait for.
template <bool ADDITIVE>
__global__ __launch_bounds__(kBlock) void eval_extras_rows_kernel(GridDesc g, const DevTables *__restrict__ tab,
                                                             uint32_t first, uint32_t count, uint32_t n_gpus,
                                                             guide_extras out) {
    __shared__ GridLds s;
    stage_grid_tables(s, g, tab);
    __syncthreads();
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < count; i = stride_on(i, gridDim.x * kBlock, count)) {
        const Candidate c = decode_index(s, g, first + i);
        const HwRecip hw = s.hw[c.hw];
        const Coef cf = make_coef(s.models[c.model], c.kn.p, c.kn.wbits);
        const uint32_t dp = n_gpus / c.kn.p;
        const double n = (double)(c.kn.s_out - 1);
        double tok_s = 0.0, tok_s1 = 0.0;
        if (c.kn.s_out > 1 && (out.cluster_tok_s || out.paper_tok_s)) {
            const TimeCoef tc = make_time_coef(cf, hw.r_peak, hw.r_bw, hw.r_link, hw.lat);
            tok_s = (double)c.kn.b * n / decode_time<ADDITIVE>(tc, c.kn.b, c.kn.s_in, c.kn.s_out - 1);
            if (out.paper_tok_s) {
                const Coef c1 = make_coef(s.models[c.model], 1u, c.kn.wbits);      // the same candidate on one GPU
                const TimeCoef t1 = make_time_coef(c1, hw.r_peak, hw.r_bw, hw.r_link, hw.lat);
                tok_s1 = (double)c.kn.b * n / decode_time<ADDITIVE>(t1, c.kn.b, c.kn.s_in, c.kn.s_out - 1);
            }
        }
        const double c_avail = hw.cap - cf.w_gpu;
        const double q = floor(c_avail / ((double)c.kn.b * cf.kv_tok));
        const uint32_t s_max = !(c_avail > 0.0) ? 0u : (q >= 4294967295.0 ? 4294967295u : (uint32_t)q);
        if (out.s_max) out.s_max[i] = s_max;
        if (out.dp_max) out.dp_max[i] = dp;
        const MemResult m = memory_check(cf, hw.cap, c.kn.b, c.kn.s_in, c.kn.s_out, c.kn.blk);
        if (out.max_parallelism) out.max_parallelism[i] = (uint64_t)dp * (uint64_t)m.b_max;
        if (out.b_adj) out.b_adj[i] = c.kn.b < m.b_max ? c.kn.b : m.b_max;
        const bool long_prompt = c.kn.s_in > c.kn.mbt;
        if (out.n_sub_batches) {
            uint32_t split = c.kn.mbt / c.kn.s_in;                    // prompts per pass (0 for a long prompt)
            split = split < c.kn.b ? split : c.kn.b;
            out.n_sub_batches[i] = long_prompt ? c.kn.b : (c.kn.b + split - 1) / split;
        }
        if (out.n_segments) out.n_segments[i] = long_prompt ? (c.kn.s_in - 1) / c.kn.mbt + 1 : 1u;
        if (out.s_adj) {
            const uint32_t len = c.kn.s_in + c.kn.s_out;              // both below 2^31
            out.s_adj[i] = len < s_max ? len : s_max;
        }
        if (out.b_max_kept || out.feasible_kept || out.s_max_kept) {
            // a KV-cache reduction that keeps the fraction kv_keep of every request's entries
            const double keep = out.kv_keep == 0.0 ? 1.0 : out.kv_keep;
            const uint32_t len = c.kn.s_in + c.kn.s_out;
            const uint64_t kept = (uint64_t)ceil(keep * (double)len);
            const uint64_t tok_req = (kept + c.kn.blk - 1) / c.kn.blk * c.kn.blk;
            const double kv_req = (double)tok_req * cf.kv_tok;
            const bool room = c_avail > 0.0;
            const double qb = floor(c_avail / kv_req), qs = floor(q / keep);
            if (out.b_max_kept) out.b_max_kept[i] = !room ? 0u : (qb >= 4294967295.0 ? 4294967295u : (uint32_t)qb);
            if (out.feasible_kept) out.feasible_kept[i] = (room && (double)c.kn.b * kv_req <= c_avail) ? 1 : 0;
            if (out.s_max_kept) out.s_max_kept[i] = !room ? 0u : (qs >= 4294967295.0 ? 4294967295u : (uint32_t)qs);
        }
        if (out.cluster_tok_s) out.cluster_tok_s[i] = (double)dp * tok_s;
        if (out.paper_tok_s)
            out.paper_tok_s[i] = ((double)dp * (double)c.kn.p) * tok_s1 / (1.0 + log2((double)c.kn.p));
    }
}

static uint32_t blocks_for(uint32_t count) {
    const uint32_t need = (count - 1) / kBlock + 1;             // (count > 0)
    const uint32_t cap = device_cus() * 8;
    return need < cap ? need : cap;
}

// Cluster columns: expanded, or one index per lane?  Expanding works a value out once per tile, per (tile, block size) and per
// (tile, token budget): `parts` of them for the tile's rows.  It pays by the work that this saves, which the throughput
// columns need most of, and by the wider stores where many bytes of a row are asked for; against it stand the latency of
// its phases and, with few columns, the values that nobody asked for.  Microseconds, one index per lane / expanded:
//   all twelve columns (57 bytes)  2 x 2 15.0 / 11.8, 6 x 1 15.0 / 14.7, 5 x 6 15.0 / 9.7 (400 000 rows); 2 x 3 10.3 / 10.0,
//                                  3 x 3 10.3 / 8.3, 6 x 1 10.2 / 10.8 (250 000); 1 x 2 14.7 / 14.9 (400 000); 2 x 3 44.7 / 25.1 (1.9 million)
//   both throughputs, or 32 bytes  2 x 2 11.6 / 8.9 and 12.6 / 10.0, 6 x 1 11.7 / 10.8 and 12.6 / 11.9 (400 000)
//   one throughput                 2 x 2 9.2 / 8.2, 1 x 64 9.2 / 8.1, 1 x 6 9.3 / 10.0 (400 000), 3 x 4 6.3 / 6.0, 2 x 3 6.4 / 7.4 (250 000)
//   s_max alone                    4 x 4 7.1 / 6.2, 3 x 4 7.2 / 7.8 (400 000), 3 x 3 9.4 / 8.9, 2 x 2 9.3 / 10.7 (700 000), 2 x 3 13.7 / 14.4
//                                  (1.3 million), 18.3 / 17.1 (1.9 million), 1 x 64 26.8 / 31.5 (3 million)
static bool expand_extras(const GridDesc &g, uint32_t count, uint64_t row_bytes, const guide_extras &out) {
    const uint32_t nb = g.div[AX_BLK].d, nm = g.div[AX_MBT].d, ts = nb * nm;
    if (ts < 4) return false;
    const double parts = (double)(1 + nb + nm) / ts;
    if (row_bytes >= 32 || (out.cluster_tok_s && out.paper_tok_s)) return count >= (parts <= 1.04 ? 250000u : 400000u);
    if (out.cluster_tok_s || out.paper_tok_s) return parts <= 1.3 && count >= (parts <= 0.8 ? 250000u : 400000u);
    return parts <= 1.0 && count >= (parts <= 0.6 ? 400000u : parts <= 0.8 ? 700000u : 1800000u);
}
// Grids with wide fast axes are expanded beyond 131 072 rows (a row per lane of two blocks per compute unit): 3.6 us a row at
// a time against 4.5 - 4.8 us at 3000 to 30 000 rows, 4.3 - 4.7 against 4.7 - 5.8 us at 100 000; at 500 000 rows the kernel
// of one index per lane before took 13 - 28 us, expanded 8 - 15 us.
constexpr uint32_t kExpandWideRows = 131072;
// Tiles of a run and blocks of the launch.  Two blocks per compute unit (what the LDS of both kernels allows at 160 KB;
// three with half the runs' length: 27 against 25 us for the full grid's twelve columns), every block the same number
// of full runs, and runs of whole multiples of 64 tiles when they are that long: their rows then start on line
// boundaries of every column unless the range itself does not.  Only then are large outputs stored past the caches, which must
// merge the halves of a line that two blocks share: 1.9 million rows of 2 x 3 tiles, all columns, 25.1 us past them on whole
// lines, 38.8 past and 26.9 through them on shared ones; 6 million of 4 x 4 tiles 141 and 80 us shared.
// Few tiles of many rows are cut into slices of at least 512 rows, a block each, which works out all of the tile and writes its
// own share of the rows (cluster columns of 250 000 rows in 64 x 64 tiles: 8.6 us, with one block a tile 14.5; one index per lane 10.3).
struct ExpandPlan {
    uint32_t per_run;
    dim3 grid;                          // (blocks, slices)
    bool lines;                         // every run's rows start on a line boundary of every column of four bytes or more
};
static ExpandPlan expand_plan(const GridDesc &g, uint32_t first, uint32_t count) {
    const uint32_t nb = g.div[AX_BLK].d, nm = g.div[AX_MBT].d, ts = nb * nm, widest = nb > nm ? nb : nm;
    const uint32_t n_tiles = (first + count - 1) / ts - first / ts + 1, most = device_cus() * 2;
    const uint32_t cap = kExpandParts / widest < kExpandTiles ? kExpandParts / widest : kExpandTiles;
    const uint32_t per_block = (uint32_t)(((uint64_t)n_tiles + most - 1) / most), rounds = (per_block + cap - 1) / cap;
    uint32_t per_run = (per_block + rounds - 1) / rounds;
    if (per_run >= 64) {
        const uint32_t up = (per_run + 63) / 64 * 64;
        per_run = up <= cap ? up : per_run / 64 * 64;
    }
    const uint32_t runs = (uint32_t)(((uint64_t)n_tiles + per_run - 1) / per_run);
    uint32_t slices = 1;
    if (per_run == 1 && ts >= 1024 && 2 * runs <= most) {
        const uint32_t by_rows = ts / 512, by_blocks = most / runs;
        slices = by_rows < by_blocks ? by_rows : by_blocks;
    }
    const bool lines = (first / ts * ts - first) % 32 == 0 && (uint64_t)per_run * ts % 32 == 0;
    return ExpandPlan{per_run, dim3(runs < most ? runs : most, slices), lines};
}

static uint32_t tile_blocks(uint32_t first, uint32_t count, uint32_t ts) {
    const uint32_t n_tiles = (first + count - 1) / ts - first / ts + 1;
    // two persistent blocks per compute unit: every wave loops over several batches of 64 tiles, so the
    // stores of one batch overlap the arithmetic of the next (measured best among 1..8 blocks per CU)
    // (every block writes one top-k partial when a top-k is folded in)
    uint32_t cap = 2 * device_cus();
    cap = cap < kSelBlocks ? cap : kSelBlocks;
    const uint32_t need = (n_tiles - 1) / kBlock + 1;
    return need < cap ? need : cap;
}

// Rows sampled for a Pareto selection over the evaluated rows.
constexpr uint32_t kSampleRows = 16384;
constexpr uint64_t kStreamBytes = 64ull << 20;      // twice the 8 x 4 MB of L2: 8-byte columns that together reach it are streamed
constexpr uint32_t kRiderBlocks = kSampleRows / kBlock;     // sample blocks appended to a plain evaluation
static_assert(kRiderBlocks == kSampleBlocks, "the scratch holds one sample front per sample block");

static uint32_t n_f64_columns(const guide_metrics &out) {
    return (out.t_prefill ? 1u : 0u) + (out.t_decode ? 1u : 0u) + (out.t_batch ? 1u : 0u) + (out.decode_tok_s ? 1u : 0u) +
           (out.cost ? 1u : 0u);
}

template <bool ADDITIVE, int NB, int NM>
static void launch_tile(const GridDesc &g, const DevTables *tab, const void *tile_tables, uint32_t first,
                        uint32_t count, double re_c, double re_b, const guide_metrics &out, const FusedSelect *fs,
                        hipStream_t stream, LaunchTiming tm) {
    // fs: a top-k folded into the evaluation (the FUSED kernel) and / or rider_blocks extra blocks that take the
    // row sample of a Pareto selection
    const FusedSelect sel = fs ? *fs : FusedSelect{};
    const dim3 grid(tile_blocks(first, count, NB * NM) + sel.rider_blocks), block(kBlock);
    const TileLds *tables = (const TileLds *)tile_tables;
    // Columns that together are larger than twice the chip's L2 are stored with the streaming hint: their lines
    // would not survive in L2 until a reader comes anyway, and not keeping them there leaves the stores of the
    // launch more room (20M rows: 163 - 166 us against 178 - 179 us; 1.9M rows inside an evaluate-and-select step:
    // 17.4 against 17.8 us, the filter pass after it 13.4 against 13.1 us; smaller outputs stay cached for their readers).
    // (a kernel of its own: a run-time choice between the two kinds of store compiles to the plain one)
    const bool stream_stores = (uint64_t)count * 8 * n_f64_columns(out) >= kStreamBytes;
    auto launch = [&](auto kernel) {
        // with timing events the launch goes through the extended call, which attaches them to the dispatch
        if (tm.start)
            hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, tm.start, tm.stop, 0, g, tab, first, count, re_c, re_b, out,
                                  sel, tables);
        else
            hipLaunchKernelGGL(kernel, grid, block, 0, stream, g, tab, first, count, re_c, re_b, out, sel, tables);
    };
    if (sel.topk) launch(eval_tile_kernel<ADDITIVE, NB, NM, true, false>);
    else if (stream_stores) launch(eval_tile_kernel<ADDITIVE, NB, NM, false, true>);
    else launch(eval_tile_kernel<ADDITIVE, NB, NM, false, false>);
}

// Tile shapes with a compiled kernel (up to four values on each of the two fastest axes); other grids take
// eval_wide_kernel.
#define GUIDE_TILE_SHAPES(X)                                                                     \
    X(2, 3) X(1, 1) X(1, 2) X(1, 3) X(1, 4) X(2, 1) X(2, 2) X(2, 4) X(3, 1) X(3, 2) X(3, 3) X(3, 4) \
    X(4, 1) X(4, 2) X(4, 3) X(4, 4)

template <bool ADDITIVE>
static bool dispatch_tile(const GridDesc &g, const DevTables *tab, const void *tile_tables, uint32_t first,
                          uint32_t count, double re_c, double re_b, const guide_metrics &out, const FusedSelect *fs,
                          hipStream_t stream, uint32_t *n_blocks, LaunchTiming tm) {
    const uint32_t nb = g.div[AX_BLK].d, nm = g.div[AX_MBT].d;
#define GUIDE_TILE(NB, NM)                                                                   \
    if (nb == NB && nm == NM) {                                                              \
        launch_tile<ADDITIVE, NB, NM>(g, tab, tile_tables, first, count, re_c, re_b, out, fs, stream, tm); \
        if (n_blocks) *n_blocks = tile_blocks(first, count, NB * NM);                        \
        return true;                                                                         \
    }
    GUIDE_TILE_SHAPES(GUIDE_TILE)
#undef GUIDE_TILE
    return false;
}

bool eval_grid_can_fuse(const GridDesc &g) {
    const uint32_t nb = g.div[AX_BLK].d, nm = g.div[AX_MBT].d;
#define GUIDE_TILE(NB, NM) if (nb == NB && nm == NM) return true;
    GUIDE_TILE_SHAPES(GUIDE_TILE)
#undef GUIDE_TILE
    return false;
}

// The tile kernels deal batches of kBlock tiles (kBlock * NB * NM consecutive rows) to their blocks round robin.
uint32_t eval_grid_row_chunk(const GridDesc &g) {
    return eval_grid_can_fuse(g) ? (uint32_t)kBlock * g.div[AX_BLK].d * g.div[AX_MBT].d : 0u;
}

size_t tile_tables_bytes() { return sizeof(TileLds); }

hipError_t launch_tile_tables(const GridDesc &g, const DevTables *tab, void *tile_tables, hipStream_t stream) {
    hipLaunchKernelGGL(tile_tables_kernel, dim3(1), dim3(kBlock), 0, stream, g, tab, (TileLds *)tile_tables);
    return hipGetLastError();
}

hipError_t launch_eval_grid_fused(const GridDesc &g, const DevTables *tab, const void *tile_tables, uint32_t first,
                                  uint32_t count, double e_c, double e_b, bool additive, const guide_metrics &out,
                                  const FusedSelect &fs, hipStream_t stream, uint32_t *n_blocks, LaunchTiming tm) {
    const double re_c = 1.0 / e_c, re_b = 1.0 / e_b;
    FusedSelect sel = fs;
    sel.rider_blocks = fs.pareto ? kRiderBlocks : 0u;
    const bool done =
        additive ? dispatch_tile<true>(g, tab, tile_tables, first, count, re_c, re_b, out, &sel, stream, n_blocks, tm)
                 : dispatch_tile<false>(g, tab, tile_tables, first, count, re_c, re_b, out, &sel, stream, n_blocks, tm);
    return done ? hipGetLastError() : hipErrorNotSupported;
}

hipError_t launch_eval_grid(const GridDesc &g, const DevTables *tab, const void *tile_tables, uint32_t first,
                            uint32_t count, double e_c, double e_b, bool additive, const guide_metrics &out,
                            hipStream_t stream, LaunchTiming tm, const FusedSelect *sample, bool *sampled) {
    const dim3 block(kBlock);
    const double re_c = 1.0 / e_c, re_b = 1.0 / e_b;
    FusedSelect rider;
    const FusedSelect *fs = nullptr;
    if (sampled) *sampled = false;
    if (sample && sampled && eval_grid_can_fuse(g)) {
        rider = *sample;
        rider.topk = 0;
        rider.rider_blocks = kRiderBlocks;
        fs = &rider;
        *sampled = true;
    }
    if (additive ? dispatch_tile<true>(g, tab, tile_tables, first, count, re_c, re_b, out, fs, stream, nullptr, tm)
                 : dispatch_tile<false>(g, tab, tile_tables, first, count, re_c, re_b, out, fs, stream, nullptr, tm))
        return hipGetLastError();
    if (count <= kExpandWideRows) {
        const dim3 rows((count + kBlock - 1) / kBlock);
        auto launch = [&](auto kernel) {
            const TileLds *tables = (const TileLds *)tile_tables;
            if (tm.start)
                hipExtLaunchKernelGGL(kernel, rows, block, 0, stream, tm.start, tm.stop, 0, g, first, count, re_c, re_b, out, tables);
            else
                hipLaunchKernelGGL(kernel, rows, block, 0, stream, g, first, count, re_c, re_b, out, tables);
        };
        if (additive) launch(eval_wide_rows_kernel<true>);
        else launch(eval_wide_rows_kernel<false>);
        return hipGetLastError();
    }
    const ExpandPlan plan = expand_plan(g, first, count);
    const bool stream_stores = plan.lines && (uint64_t)count * 8 * n_f64_columns(out) >= kStreamBytes;
    auto launch = [&](auto kernel) {
        const TileLds *tables = (const TileLds *)tile_tables;
        if (tm.start)
            hipExtLaunchKernelGGL(kernel, plan.grid, block, 0, stream, tm.start, tm.stop, 0, g, first, count, re_c, re_b,
                                  out, tables, plan.per_run);
        else
            hipLaunchKernelGGL(kernel, plan.grid, block, 0, stream, g, first, count, re_c, re_b, out, tables,
                               plan.per_run);
    };
    if (additive && stream_stores) launch(eval_wide_kernel<true, true>);
    else if (additive) launch(eval_wide_kernel<true, false>);
    else if (stream_stores) launch(eval_wide_kernel<false, true>);
    else launch(eval_wide_kernel<false, false>);
    return hipGetLastError();
}

hipError_t launch_eval_extras(const GridDesc &g, const DevTables *tab, uint32_t first, uint32_t count, uint32_t n_gpus,
                              bool additive, const guide_extras &out, hipStream_t stream) {
    auto bytes = [](const void *p, uint64_t width) { return p ? width : 0; };
    const uint64_t per_row = bytes(out.s_max, 4) + bytes(out.dp_max, 4) + bytes(out.max_parallelism, 8) + bytes(out.cluster_tok_s, 8) +
                             bytes(out.paper_tok_s, 8) + bytes(out.b_adj, 4) + bytes(out.n_sub_batches, 4) +
                             bytes(out.n_segments, 4) + bytes(out.s_adj, 4) + bytes(out.b_max_kept, 4) + bytes(out.s_max_kept, 4);
    if (!expand_extras(g, count, per_row, out)) {
        const dim3 grid(blocks_for(count)), block(kBlock);
        if (additive)
            hipLaunchKernelGGL(eval_extras_rows_kernel<true>, grid, block, 0, stream, g, tab, first, count, n_gpus, out);
        else
            hipLaunchKernelGGL(eval_extras_rows_kernel<false>, grid, block, 0, stream, g, tab, first, count, n_gpus, out);
        return hipGetLastError();
    }
    const ExpandPlan plan = expand_plan(g, first, count);
    const bool stream_stores = plan.lines && count * per_row >= kStreamBytes;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, plan.grid, dim3(kBlock), 0, stream, g, tab, first, count, n_gpus, out, plan.per_run);
    };
    if (additive && stream_stores) launch(eval_extras_kernel<true, true>);
    else if (additive) launch(eval_extras_kernel<true, false>);
    else if (stream_stores) launch(eval_extras_kernel<false, true>);
    else launch(eval_extras_kernel<false, false>);
    return hipGetLastError();
}

hipError_t launch_eval_sweep(const GridDesc &g, const DevTables *tab, const void *tile_tables, uint32_t first,
                             uint32_t count, uint32_t n_eff, bool additive, const guide_stats &out, hipStream_t stream) {
    const uint32_t ts = g.div[AX_BLK].d * g.div[AX_MBT].d, nm = g.div[AX_MBT].d;
    const uint32_t most = 2 * device_cus();                     // resident blocks: two per compute unit
    SweepItems items;
    items.inner = g.div[AX_TP].d * g.div[AX_WBITS].d;
    const uint32_t span = items.inner * g.div[AX_SOUT].d;       // tiles of a setting of the axes above s_out
    items.first_group = first / ts / span;
    const uint32_t n_rest = ((first + count - 1) / ts - first / ts + 1) * nm;
    items.prefill_end = ((first + count - 1) / ts / span - items.first_group + 1) * items.inner * nm;
    // Items of the prefill pay where they are few (six values of s_out or more), the others fill the chip more than once, and there
    // are samples enough to sort.  In us, all columns by one item / apart, 64 samples: 1.9 million rows 142 / 122, additive 99 / 80,
    // without columns of the prefill 136 / 117; 950 000 75.4 / 63.3; 317 000 32.6 / 26.9; seven values of s_out 116 / 103, six 99 / 89.
    // 1.9 million rows of two samples 54.2 / 56.7 (without columns of the prefill 52.6 / 54.3), of three 60.6 / 60.6 - 62.0, of four
    // 63.4 / 63.6 - 65.5, additive 40.4 / 38.7, 950 000 38.0 / 36.2; of five 64.6 / 64.6, of eight 60.2 / 58.2, of 24 79.3 / 74.4 (with few
    // samples stores are half of it, and where the columns lie makes a difference of 2 us).  The lines of lengths and rows are on the safe side: five values
    // 89 / 78, four 76 / 71, 127 000 rows (half a round) 18.9 / 17.1.
    const bool shared = n_eff >= 4 && n_rest > most * kBlock && items.prefill_end < n_rest / 5 && n_rest < 3u << 30;      // (the sum fits 32 bits)
    items.n_prefill = shared ? (items.prefill_end - 1) / kWave * kWave + kWave : 0u;
    items.n = items.n_prefill + n_rest;
    const uint32_t need = (items.n - 1) / kBlock + 1;
    const dim3 grid(need < most ? need : most), block(kBlock);
    const TileLds *tables = (const TileLds *)tile_tables;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, g, tab, first, count, n_eff, out, tables, items); };
    if (additive && shared) launch(eval_sweep_kernel<true, true>);
    else if (additive) launch(eval_sweep_kernel<true, false>);
    else if (shared) launch(eval_sweep_kernel<false, true>);
    else launch(eval_sweep_kernel<false, false>);
    return hipGetLastError();
}

}  // namespace guide
