// Random-sampled configuration space: candidate i is drawn from a counter-based
// generator keyed by (seed, i), evaluated, and folded into reduced outputs
// (feasible count, per model-size bucket best candidate, latency histogram)
// inside the kernel.  Only a few KB leave the chip.
#include "kernels.hpp"
#include "perf_model.hpp"
#include "reduce.hpp"

namespace guide {

namespace {

constexpr uint32_t kMaxBuckets = GUIDE_MAX_BUCKET_EDGES + 1;

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each two
// 64x64 -> 128 bit multiplies by the published constants; the key advances by
// the Weyl increments between rounds.
struct Block256 {
    uint64_t v[4];
};
// The two words of a 64 x 64 bit product by four 32-bit multiply-adds, the low word from the same ones as the high word.
__device__ inline void mul128(uint64_t m, uint64_t x, uint64_t &hi, uint64_t &lo) {
    const uint32_t m0 = (uint32_t)m, m1 = (uint32_t)(m >> 32), x0 = (uint32_t)x, x1 = (uint32_t)(x >> 32);
    const uint64_t p = (uint64_t)m0 * x0;
    const uint64_t t = (uint64_t)m1 * x0 + (p >> 32);
    const uint64_t u = (uint64_t)m0 * x1 + (uint32_t)t;
    hi = (uint64_t)m1 * x1 + (t >> 32) + (u >> 32);
    lo = (u << 32) | (uint32_t)p;
}
__device__ inline uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {       // one instruction per half
    const uint32_t lo = __builtin_amdgcn_bitop3_b32((uint32_t)a, (uint32_t)b, (uint32_t)c, 0x96);
    const uint32_t hi = __builtin_amdgcn_bitop3_b32((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), 0x96);
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline Block256 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0, uint64_t k1) {
    constexpr uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    constexpr uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t hi0, lo0, hi1, lo1;
        mul128(M0, c0, hi0, lo0);
        mul128(M1, c2, hi1, lo1);
        const uint64_t n0 = xor3(hi1, c1, k0), n2 = xor3(hi0, c3, k1);
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += W0; k1 += W1;
    }
    Block256 b;
    b.v[0] = c0; b.v[1] = c1; b.v[2] = c2; b.v[3] = c3;
    return b;
}

constexpr uint32_t kSampledBlock = 512;         // threads of a block: two blocks of a compute unit share its LDS

// Every table as the 64-bit number that the model computes with: a conversion per candidate costs as much as a multiplication.
struct SampledLds {
    double d[GUIDE_LATTICE], batch[GUIDE_LATTICE], s_in[GUIDE_LATTICE], s_out[GUIDE_LATTICE];  // d: heads x 128
    double r_sin_up[GUIDE_LATTICE], op[GUIDE_LATTICE], r_bw[GUIDE_LATTICE];                    // op: seconds per two operations
    uint64_t win_key[kSampledBlock / kWave][kMaxBuckets], win_idx[kSampledBlock / kWave][kMaxBuckets];
    double edges[kMaxBuckets];                                   // ascending, the unused ones no number
    uint32_t hist[GUIDE_HIST_BINS];
    // the small tables, with the reciprocals of what is divided by (nudged for floor division but for 1 / tp)
    double cap[8], tp[4], r_tp[4], r_tp_up[4], weight_bytes[4], blk[2], r_blk[2], mbt[4], r_mbt[4], d_kv[4];    // d_kv: 0: as many as heads
};
static_assert(kMaxBuckets == 16, "the search over the edges takes four steps");

// Block partials: [block][bucket] keys and rows of the bucket winners, histograms, feasible candidates.
struct SampledScratch {
    uint64_t key[kSampledMaxBlocks][kMaxBuckets];
    uint64_t idx[kSampledMaxBlocks][kMaxBuckets];
    uint32_t hist[kSampledMaxBlocks][GUIDE_HIST_BINS];
    uint32_t feasible[kSampledMaxBlocks];
};

// 16-bit field j of the block (lowest field of word 0 first).
__device__ inline uint32_t field(const Block256 &b, int j) { return (uint32_t)(b.v[j >> 2] >> (16 * (j & 3))) & 0xFFFFu; }

// floor(x / y) of whole numbers below 2^47, from the nudged reciprocal of y
__device__ inline double floor_by(double x, double r_up) { return floor(x * r_up); }

// Pass times of a dense model whose heads are 128 wide (so that query and model widths are equal).  Every linear task is a
// matrix of X elements: 2 X operations and `bytes` X weight bytes, and A activation bytes a token.  X and A times tp are whole numbers;
// seconds per operation and per byte, with 1 / tp in them, come in with a pass's token count.
struct DenseTimes {
    double X[4], XW[4], A[4];               // qkv, output, up and gate, down
    double X_lm, XW_lm, A_lm;
    double op, byte;                        // seconds per two operations and per byte, over tp
    double lin;                             // norms and all-reduces: seconds per token
    double c_att, m_att_t, m_att_k;         // attention: per query-context pair, per token, per cached token
};
__device__ inline DenseTimes dense_times(double d, double dkv, double dff, double V, double p, double weight_bytes, double kv_bytes,
                                         double rp, double op, double r_bw, double link_div) {
    DenseTimes t;
    t.op = op * rp;
    t.byte = r_bw * rp;
    const double d2 = d + d, G = d2 * p, wb = weight_bytes * t.byte, f1 = d * dff;
    t.X[0] = d * fma(2.0, dkv, d);
    t.X[1] = d * d;
    t.X[2] = f1 + f1;
    t.X[3] = f1;
    t.A[0] = G + fma(4.0, dkv, d2);
    t.A[1] = G + d2;
    t.A[2] = fma(4.0, dff, G);
    t.A[3] = fma(2.0, dff, G);
    t.X_lm = d * V;
    t.A_lm = fma(2.0, V, G);
#pragma unroll
    for (int i = 0; i < 4; ++i) t.XW[i] = t.X[i] * wb;
    t.XW_lm = t.X_lm * wb;
    t.lin = fma(4.0 * G, t.byte, (4.0 * (p - 1.0)) * d2 * (link_div * t.byte));       // (no transfers for p = 1)
    t.c_att = d2 * t.op;
    t.m_att_t = 4.0 * d * t.byte;
    t.m_att_k = kv_bytes * r_bw;
    return t;
}
// One layer without attention for a pass of T tokens.
template <bool ADDITIVE>
__device__ inline double dense_layer(const DenseTimes &t, double T) {
    const double ops = T * t.op, bytes = T * t.byte;
    double s = T * t.lin;
    if (ADDITIVE) {
        const double X = (t.X[0] + t.X[1]) + (t.X[2] + t.X[3]), A = (t.A[0] + t.A[1]) + (t.A[2] + t.A[3]);
        return s + fma(ops, X, fma(bytes, A, (t.XW[0] + t.XW[1]) + (t.XW[2] + t.XW[3])));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) s += op_time<ADDITIVE>(t.X[i] * ops, fma(t.A[i], bytes, t.XW[i]));
    return s;
}
template <bool ADDITIVE>
__device__ inline double dense_head(const DenseTimes &t, double n) {
    return op_time<ADDITIVE>(t.X_lm * (n * t.op), fma(t.A_lm, n * t.byte, t.XW_lm));
}

// Attention of n segments of M tokens, the j-th at context M j: the sum of max(al M j, k M j + M m), al = M times the time per pair.
template <bool ADDITIVE>
__device__ inline double segment_attention(double M, double n, double al, double k, double m) {
    const double h = 0.5 * n, all = fma(n, h, h);       // 1 + .. + n
    if (ADDITIVE) return M * fma(al + k, all, n * m);
    double j = n;                                       // the last segment that is bound by reading
    if (al > k) j = fmin(floor(m * fast_recip(al - k)), n);
    const double g = 0.5 * j, low = fma(j, g, g);
    return M * fma(k, low, fma(j, m, al * (all - low)));
}

// Bound by the vector ALU: an instruction on 64-bit values takes 4.3 - 5 of a SIMD's cycles, a 64-bit reciprocal 16, and the loop
// has 507 (a third of them the generator's).  2^28 candidates: 3.59 ms a call; 4.58 ms with every task's coefficients
// divided out, long and short prompts as two paths and integer tables; a block of 256 threads instead of 512 would not
// leave room for the tables four waves a SIMD deep.  148 000 candidates 33.7 us, 49.3 us with histograms added up by atomics and a
// launch that cleared them.
// COLUMNS: some per-candidate column is asked for.
template <bool ADDITIVE, bool COLUMNS>
__global__ __launch_bounds__(kSampledBlock, 4) void eval_sampled_kernel(const SpaceTables *__restrict__ tab, uint64_t seed,
                                                              uint64_t first, uint64_t count, double ttft_cap,
                                                              guide_sampled_out out, SampledScratch *scratch) {
    __shared__ SampledLds s;
    constexpr int kWaves = kSampledBlock / kWave;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    for (uint32_t i = threadIdx.x; i < GUIDE_LATTICE; i += kSampledBlock) {
        s.d[i] = 128.0 * (double)tab->heads[i];
        s.batch[i] = (double)tab->batch[i];
        s.s_in[i] = (double)tab->s_in[i];
        s.s_out[i] = (double)tab->s_out[i];
        s.r_sin_up[i] = recip_up(1.0 / (double)tab->s_in[i]);
        s.op[i] = 2.0 * (1.0 / tab->peak[i]);
        s.r_bw[i] = 1.0 / tab->bw[i];
    }
    for (uint32_t i = threadIdx.x; i < kWaves * kMaxBuckets; i += kSampledBlock) {
        (&s.win_key[0][0])[i] = kNone;
        (&s.win_idx[0][0])[i] = kNone;
    }
    for (uint32_t i = threadIdx.x; i < GUIDE_HIST_BINS; i += kSampledBlock) s.hist[i] = 0;
    if (threadIdx.x < 8) s.cap[threadIdx.x] = tab->cap[threadIdx.x];
    if (threadIdx.x < 4) {
        const uint32_t i = threadIdx.x, p = tab->tp[i], m = max(tab->mbt[i], 1u);
        s.tp[i] = (double)p;
        s.r_tp[i] = 1.0 / (double)p;
        s.r_tp_up[i] = recip_up(1.0 / (double)p);
        s.weight_bytes[i] = (double)tab->wbits[i] * 0.125;
        s.d_kv[i] = 128.0 * (double)tab->kv_choices[i];
        s.mbt[i] = (double)tab->mbt[i];
        s.r_mbt[i] = recip_up(1.0 / (double)m);
    }
    if (threadIdx.x < 2) {
        s.blk[threadIdx.x] = (double)tab->kv_block[threadIdx.x];
        s.r_blk[threadIdx.x] = recip_up(1.0 / (double)tab->kv_block[threadIdx.x]);
    }
    if (threadIdx.x < kWave) {                          // a bucket is a number of edges, whatever their order
        const double e = lane < GUIDE_MAX_BUCKET_EDGES && lane < (int)tab->n_edges ? tab->edges[lane] : INFINITY;
        const double mine = e == e ? e : INFINITY;
        uint32_t rank = 0;
#pragma unroll
        for (int j = 0; j < (int)kMaxBuckets; ++j) {
            const double other = __shfl(mine, j, kWave);
            rank += other < mine || (other == mine && j < lane) ? 1u : 0u;
        }
        if (lane < (int)kMaxBuckets) s.edges[rank] = mine < INFINITY ? mine : __builtin_nan("");
    }
    __syncthreads();
    bool p_exact = true;                                // every tp is a power of two (uniform)
    for (int i = 0; i < 4; ++i) p_exact = p_exact && (tab->tp[i] & (tab->tp[i] - 1)) == 0;
    const uint32_t layers_lo = tab->layers_lo, layers_n = tab->layers_n;
    const double V = (double)tab->vocab;
    const uint64_t ffn_lo = (uint64_t)tab->ffn_lo_x2 * 65536u, ffn_span = tab->ffn_span_x2;
    // feed-forward widths fit 32 bits, and the products that they come from 53 (uniform)
    const bool ffn_exact = tab->ffn_lo_x2 < (1u << 15) && tab->ffn_span_x2 < (1u << 15);
    const uint32_t n_edges = tab->n_edges;
    const double link_div = tab->link_div;
    const uint64_t stride = (uint64_t)gridDim.x * kSampledBlock;
    const uint64_t iters = (count + stride - 1) / stride;   // same trip count for every lane
    for (uint64_t it = 0; it < iters; ++it) {
        const uint64_t i = it * stride + (uint64_t)blockIdx.x * kSampledBlock + threadIdx.x;
        const bool live = i < count;
        bool feasible = false, wins = false;
        Pair cand = {kNone, kNone};
        uint32_t bucket = 0;
        if (live) {
            const uint64_t id = first + i;
            const Block256 r = philox4x64_10(id, 0, 0, 0, seed, 0);
            const double L = (double)(layers_lo + ((field(r, 0) * layers_n) >> 16));
            const double d = s.d[field(r, 1) >> 6], some_kv = s.d_kv[field(r, 2) >> 14], dkv = some_kv != 0.0 ? some_kv : d;
            // d_ff = 128 * floor(ratio * n_h + 1/2), ratio = (lo_x2 + span_x2 * u / 65536) / 2
            double dff;
            if (ffn_exact)
                dff = 128.0 * floor(fma(fma((double)field(r, 3), (double)ffn_span, (double)ffn_lo), d * 0x1p-24, 0.5));
            else
                dff = (double)(128u * (uint32_t)(((ffn_lo + ffn_span * field(r, 3)) * (uint64_t)(d * 0x1p-7) + 65536u) >> 17));
            const uint32_t i_sin = field(r, 8) >> 6, i_tp = field(r, 10) >> 14, i_blk = field(r, 12) >> 15, i_mbt = (field(r, 13) * 3u) >> 16;
            const double b = s.batch[field(r, 7) >> 6], S = s.s_in[i_sin], o = s.s_out[field(r, 9) >> 6];
            const double p = s.tp[i_tp], rp = s.r_tp[i_tp], weight_bytes = s.weight_bytes[(field(r, 11) * 3u) >> 16];
            const double blk = s.blk[i_blk], M = s.mbt[i_mbt], r_mbt = s.r_mbt[i_mbt];
            const double op = s.op[field(r, 4) >> 6], r_bw = s.r_bw[field(r, 5) >> 6], cap = s.cap[(field(r, 6) * 6u) >> 16];

            // bytes of a cached token and layer; KV heads replicate when there are fewer than tp
            const double kv_bytes = 512.0 * floor_by(fma(dkv, 0x1p-7, p - 1.0), s.r_tp_up[i_tp]);
            const DenseTimes t = dense_times(d, dkv, dff, V, p, weight_bytes, kv_bytes, rp, op, r_bw, link_div);

            // memory (all but the division by tp whole numbers)
            const double p_total = fma(L, fma(2.0 * d, d + dkv, 3.0 * t.X[3]), 2.0 * t.X_lm);
            const double w_total = weight_bytes * p_total, w_gpu = p_exact ? w_total * rp : w_total / p;
            const double c_avail = cap - w_gpu;
            const double kv_req = floor_by(S + o + (blk - 1.0), s.r_blk[i_blk]) * blk * (L * kv_bytes);
            feasible = c_avail > 0.0 && b * kv_req <= c_avail;

            // Prefill: two kinds of passes.  Prompts that fit the budget: n passes of R of them, then one of the rest.  Longer
            // ones, one request after another: n segments of mbt tokens, then the last tokens with the LM head.
            const double R = fmin(floor_by(M, s.r_sin_up[i_sin]), b);
            double n = R < b ? floor_by(b, recip_up(fast_recip(R))) : 1.0, rem = fma(-n, R, b);
            double T_A = R * S, T_B = rem * S, head = R, heads = n, scale = 1.0;
            double att = S * op_time<ADDITIVE>(S * t.c_att, t.m_att_k + t.m_att_t);        // of one prompt
            const bool seg = S > M, two = seg || rem > 0.0;
            if (seg) {
                n = floor_by(S + (M - 1.0), r_mbt) - 1.0;
                T_A = M;
                T_B = fma(-n, M, S);
                rem = 0.0;
                head = heads = 1.0;
                scale = b;
                att = segment_attention<ADDITIVE>(M, n, M * t.c_att, t.m_att_k, t.m_att_t) +
                      op_time<ADDITIVE>(T_B * S * t.c_att, fma(S, t.m_att_k, T_B * t.m_att_t));
            }
            double layer_times = n * dense_layer<ADDITIVE>(t, T_A), head_times = heads * dense_head<ADDITIVE>(t, head);
            if (two) layer_times += dense_layer<ADDITIVE>(t, T_B);
            if (rem > 0.0) head_times += dense_head<ADDITIVE>(t, rem);
            const double t_prefill = fma(L, fma(scale, layer_times, b * att), scale * head_times);

            // decode: s_out - 1 steps of b tokens
            const double steps = o - 1.0;
            double t_decode = 0.0;
            if (steps > 0.0) {
                const double series = attention_series<ADDITIVE>(t.c_att, t.m_att_k, t.m_att_t, S, 1.0, 1.0, steps);
                t_decode = fma(L, fma(steps, dense_layer<ADDITIVE>(t, b), b * series), steps * dense_head<ADDITIVE>(t, b));
            }
            const double t_batch = t_prefill + t_decode;
            const double spent = p * (1.0e6 / 3600.0) * t_batch, made = b * o;

            uint32_t at = 0;                                        // in bytes
#pragma unroll
            for (uint32_t step = 64; step >= 8; step >>= 1)
                at |= p_total >= *(const double *)((const char *)s.edges + at + step - 8) ? step : 0u;
            bucket = at / 8;
            if (feasible) {
                // 8 bins per octave from the exponent and the top three mantissa bits
                int bin = (int)((uint32_t)(__double_as_longlong(t_batch) >> 32) >> 17) - ((1023 - 12) << 3);
                bin = bin < 0 ? 0 : (bin > GUIDE_HIST_BINS - 1 ? GUIDE_HIST_BINS - 1 : bin);
                atomicAdd(&s.hist[bin], 1u);
                // the bucket's best so far (no number at first: passes); a candidate that is not near it saves the division
                const double best = __longlong_as_double((long long)(s.win_key[wave][bucket] & 0x7FFFFFFFFFFFFFFFull));
                wins = t_prefill <= ttft_cap && !(spent > best * made * (1.0 + 0x1p-40));
            }
            if (COLUMNS || wins) {
                const double cost = spent * fast_recip(made);
                wins = wins && cost == cost;
                cand.key = key_of(cost);
                cand.idx = id;
                if (COLUMNS) {
                    if (out.t_prefill) out.t_prefill[i] = t_prefill;
                    if (out.t_batch) out.t_batch[i] = t_batch;
                    if (out.cost) out.cost[i] = cost;
                    if (out.b_max) {
                        const double q = floor(c_avail / kv_req);
                        out.b_max[i] = !(c_avail > 0.0) ? 0u : (q >= 4294967295.0 ? 4294967295u : (uint32_t)q);
                    }
                    if (out.feasible) out.feasible[i] = feasible ? 1 : 0;
                    if (out.bucket) out.bucket[i] = bucket;
                }
            }
        }
        if (__ballot(wins)) slot_update(s.win_key[wave], s.win_idx[wave], bucket, wins, cand);
    }
    __syncthreads();
    static_assert(GUIDE_HIST_BINS % kWave == 0 && GUIDE_HIST_BINS <= kSampledBlock, "whole waves take a bin per lane");
    if (threadIdx.x < GUIDE_HIST_BINS) scratch->hist[blockIdx.x][threadIdx.x] = s.hist[threadIdx.x];
    if (threadIdx.x < kWave) {                          // every feasible candidate is in a bin
        uint32_t n = 0;
#pragma unroll
        for (uint32_t q = 0; q < GUIDE_HIST_BINS / kWave; ++q) n += s.hist[q * kWave + lane];
        n = wave_sum(n);                                // (a block's candidates: fewer than 2^32)
        if (lane == 0) scratch->feasible[blockIdx.x] = n;
    }
    for (uint32_t b = threadIdx.x; b <= n_edges; b += kSampledBlock) {
        Pair best = {s.win_key[0][b], s.win_idx[0][b]};
        for (int wv = 1; wv < kWaves; ++wv) {
            const Pair o = {s.win_key[wv][b], s.win_idx[wv][b]};
            best = pair_min(best, o);
        }
        scratch->key[blockIdx.x][b] = best.key;
        scratch->idx[blockIdx.x][b] = best.idx;
    }
}

// Second pass: the first kFinalHist blocks add up the histograms, kFinalBins bins each (summed in global memory, the
// 512 blocks of a long call take turns at five cache lines for 8 us and more), the others take a bucket each:
// least (cost, index) over the block partials.
constexpr uint32_t kFinalThreads = 256, kFinalBins = 16, kFinalHist = GUIDE_HIST_BINS / kFinalBins;
__global__ __launch_bounds__(kFinalThreads) void sampled_final_kernel(const SampledScratch *__restrict__ scratch,
                                                                      uint32_t n_blocks, guide_sampled_out out) {
    constexpr uint32_t kRows = kFinalThreads / kFinalBins, kWaves = kFinalThreads / kWave;
    __shared__ uint64_t s_sum[kRows][kFinalBins];
    __shared__ Pair s_best[kWaves];
    const uint32_t t = threadIdx.x;
    if (blockIdx.x < kFinalHist) {
        const uint32_t bin = t % kFinalBins, row = t / kFinalBins;
        uint64_t n = 0;
#pragma unroll 8
        for (uint32_t i = row; i < n_blocks; i += kRows) n += scratch->hist[i][blockIdx.x * kFinalBins + bin];
        s_sum[row][bin] = n;
        __syncthreads();
        if (t < kFinalBins) {
            n = 0;
            for (uint32_t r = 0; r < kRows; ++r) n += s_sum[r][t];
            out.hist[blockIdx.x * kFinalBins + t] = n;
        }
        return;
    }
    const uint32_t b = blockIdx.x - kFinalHist;
    Pair best = {kNone, kNone};
    uint64_t n = 0;
    for (uint32_t i = t; i < n_blocks; i += kFinalThreads) {
        const Pair o = {scratch->key[i][b], scratch->idx[i][b]};
        best = pair_min(best, o);
        n += scratch->feasible[i];
    }
    best = wave_min(best);
    if (t % kWave == 0) s_best[t / kWave] = best;
    if (b == 0) {                                       // (block-uniform)
        for (int off = kWave / 2; off > 0; off >>= 1) n += __shfl_xor(n, off, kWave);
        if (t % kWave == 0) s_sum[0][t / kWave] = n;
    }
    __syncthreads();
    if (t == 0) {
        for (uint32_t w = 1; w < kWaves; ++w) best = pair_min(best, s_best[w]);
        out.win_idx[b] = best.idx;
        out.win_val[b] = best.idx == kNone ? INFINITY : value_of(best.key);
        if (b == 0) {
            n = 0;
            for (uint32_t w = 0; w < kWaves; ++w) n += s_sum[0][w];
            out.feasible_count[0] = n;
        }
    }
}

}  // namespace

size_t sampled_scratch_bytes() { return sizeof(SampledScratch); }

hipError_t launch_eval_sampled(const SpaceTables *tab, uint64_t seed, uint64_t first, uint64_t count, double ttft_cap,
                               bool additive, const guide_sampled_out &out, void *scratch, hipStream_t stream,
                               uint32_t n_edges) {
    uint64_t need = (count + kSampledBlock - 1) / kSampledBlock;
    if (need == 0) need = 1;
    // two blocks of each of 256 compute units are resident; enough of them, on any part of a chip, that one has fewer than 2^32 of
    // 2^40.  (No room for more of them: a context is made and destroyed in 65 us with up to 1 MB of partials, in 110 us beyond.)
    const uint32_t nb = (uint32_t)(need < kSampledMaxBlocks ? need : kSampledMaxBlocks);
    SampledScratch *sc = (SampledScratch *)scratch;
    const bool columns = out.t_prefill || out.t_batch || out.cost || out.b_max || out.feasible || out.bucket;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nb), dim3(kSampledBlock), 0, stream, tab, seed, first, count, ttft_cap, out, sc);
    };
    if (additive && columns) launch(eval_sampled_kernel<true, true>);
    else if (additive) launch(eval_sampled_kernel<true, false>);
    else if (columns) launch(eval_sampled_kernel<false, true>);
    else launch(eval_sampled_kernel<false, false>);
    hipLaunchKernelGGL(sampled_final_kernel, dim3(kFinalHist + n_edges + 1), dim3(kFinalThreads), 0, stream, (const SampledScratch *)sc, nb,
                       out);
    return hipGetLastError();
}

}  // namespace guide
