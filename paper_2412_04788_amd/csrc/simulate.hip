// Step-level continuous-batching simulation, one serving configuration per
// lane, and the per-configuration TTFT percentiles.
//
// The paper states that the frameworks' dynamic batching and split flow are
// simulated (Overview) without giving the procedure; the scheduler simulated
// here is documented in guide.h.  The engine state is kept in aggregated form:
//   - admission is FCFS, so admitted requests are the index range [.., next);
//   - prompt chunks are handed out in admission order, so at most the head of
//     the prefill queue [comp, next) is partially prefilled;
//   - a request that finished its prompt decodes on every later step, so its
//     finishing step is known when its prompt completes: decoders live in a
//     per-lane 4-ary min-heap keyed by finishing step (root in registers, the
//     rest in LDS as far as it goes), and their number and total context are
//     two running numbers.
// A request therefore costs a few pass-time evaluations and O(log n) heap
// traffic; the steps in between cost an addition to the clock or less.
#include <type_traits>

#include "kernels.hpp"
#include "perf_model.hpp"
#include "reduce.hpp"

namespace guide {

namespace {

constexpr uint32_t kSimBlock = 256;      // one block per compute unit: the trace is staged once, the rest of LDS holds heaps
constexpr uint32_t kPctBlock = 256;
constexpr size_t kSimStaticLds = 64;     // the simulation kernel's own static LDS (wave totals)

struct RequestsLds {
    double arrival[GUIDE_MAX_REQUESTS];      // at unit rate
    uint2 len[GUIDE_MAX_REQUESTS];           // prompt and generated tokens
};

constexpr uint32_t kHeapWidth = 4;     // children per heap node
constexpr uint32_t kKeyBins = 1024;      // buckets of the expected-concurrency ordering
// Lists are ordered where that saves more than its four launches (17 us): from 16 requests on, and when lanes share a
// wave at all.  Ordered / as given, in us: 2000 x 8 101 / 85, 5000 x 8 136 / 129, 5000 x 16 193 / 203, 65 536 x 16 571 / 576,
// 5000 x 32 352 / 396, 20 000 x 128 1200 / 1446 (stepped); 65 536 x 16 541 / 526, 5000 x 32 279 / 289 (closed form); one lane
// per wave: the same 636 with 128 requests, and 31 / 13 for one configuration.
constexpr uint32_t kOrderRequests = 16;

// Workspace: heap[position][node] (u64 keys), first[cfg][req] and fin[cfg][req] (time of the first and of the
// last token), then the launch order: perm[position] = configuration, bucket of each configuration, bucket counters.
struct SimWs {
    uint64_t *heap;
    double *first, *fin;
    uint32_t *perm;
    uint32_t *bucket;     // [n_cfg]: bucket of each configuration
    uint32_t *bins;       // [kKeyBins]: counts, then scatter cursors
};
SimWs sim_ws(void *ws, uint32_t n_cfg, uint32_t n_req) {
    SimWs w;
    w.heap = (uint64_t *)ws;
    w.first = (double *)(w.heap + (size_t)n_cfg * n_req);
    w.fin = w.first + (size_t)n_cfg * n_req;
    w.perm = (uint32_t *)(w.fin + (size_t)n_cfg * n_req);
    w.bucket = w.perm + n_cfg;
    w.bins = w.bucket + n_cfg;
    return w;
}

// Grid index -> axis values (s_in / s_out digits are decoded but unused by the simulator).
__device__ inline bool decode_sim_index(const uint32_t (*axis)[GUIDE_MAX_AXIS_VALUES], const GridDesc &g, uint32_t idx,
                                        uint32_t *v) {
    uint32_t rem = idx;
#pragma unroll
    for (int a = kNumAxes - 1; a > 0; --a) {
        const uint32_t q = div32(rem, g.div[a]);
        v[a] = axis[a][rem - q * g.div[a].d];
        rem = q;
    }
    const bool bad = rem >= g.div[0].d;
    v[0] = axis[0][bad ? 0 : rem];
    return bad;
}

// Lanes of a wave run until their slowest configuration ends, and a lane's heap wants as much LDS as it has
// sequences running, so configurations are ordered by an estimate of their concurrency: Little's law (arrival
// rate x latency), with the latency at that concurrency, clamped to [1, what the sequence cap and the KV pool let
// in].  Buckets of a hundredth of an octave.  Only the order and the shares of LDS depend on it, never a result.
__device__ inline uint32_t bucket_of(float conc) {
    const int k = (int)(__log2f(fmaxf(conc, 1.0f)) * 100.0f);
    return (uint32_t)(k > (int)kKeyBins - 1 ? (int)kKeyBins - 1 : k);
}
__device__ inline float expected_of(uint32_t bucket) { return exp2f((float)bucket * 0.01f); }
// Counting and scattering go through a histogram per block in LDS: the buckets in use are few, and one global atomic
// per configuration serialises on them (197 + 195 us for 65 536 configurations).
constexpr uint32_t kOrderBlock = 1024;
static_assert(kOrderBlock == kKeyBins, "a thread per bucket");
template <bool ADDITIVE>
__global__ __launch_bounds__(kOrderBlock) void sim_order_count_kernel(GridDesc g, const DevTables *__restrict__ tab,
                                                                      uint32_t n_req,
                                                                      const uint32_t *__restrict__ cfg_idx,
                                                                      const double *__restrict__ rate_in, uint32_t n_cfg,
                                                                      SimWs ws, double sum_in, double sum_out) {
    __shared__ uint32_t s_n[kKeyBins];
    s_n[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t c = blockIdx.x * kOrderBlock + threadIdx.x;
    if (c < n_cfg) {
        uint32_t v[kNumAxes];
        const bool bad = decode_sim_index(tab->axis_vals, g, cfg_idx[c], v);
        uint32_t b = 0;
        const double rate = rate_in[c];
        if (!bad && rate > 0.0) {
            const guide_hw hw = tab->hw[v[AX_HW]];
            const Coef cf = make_coef(tab->models[v[AX_MODEL]], v[AX_TP], v[AX_WBITS]);
            const TimeCoef tc = make_time_coef(cf, 1.0 / hw.peak_flops, 1.0 / hw.hbm_bw, 1.0 / hw.link_bw, hw.link_lat);
            const double mean_in = sum_in / (double)n_req, mean_out = sum_out / (double)n_req;
            const double ctx = mean_in + 0.5 * mean_out;
            const double pool = floor(fmax(hw.cap_bytes - cf.w_gpu, 0.0) / ((mean_in + mean_out + 0.5 * (double)v[AX_BLK]) * cf.kv_tok));
            const double most = fmin(fmin((double)v[AX_BATCH], (double)n_req), fmax(pool, 1.0));
            // twice the share of time that prompts take holds the decoders up
            const double busy = fmin(2.0 * rate * pass_time<ADDITIVE>(tc, mean_in, mean_in * mean_in, mean_in, 1.0), 0.95);
            double conc = 1.0;
            for (int it = 0; it < 8; ++it)
                conc = fmin(fmax(rate * mean_out * pass_time<ADDITIVE>(tc, conc, conc * ctx, conc * ctx, conc) / (1.0 - busy), 1.0), most);
            b = bucket_of((float)conc);
        }
        ws.bucket[c] = b;
        atomicAdd(&s_n[b], 1u);
    }
    __syncthreads();
    if (s_n[threadIdx.x]) atomicAdd(&ws.bins[threadIdx.x], s_n[threadIdx.x]);
}

__global__ __launch_bounds__(kKeyBins) void sim_order_scan_kernel(SimWs ws) {
    __shared__ uint32_t s[kKeyBins];
    const uint32_t t = threadIdx.x;
    s[t] = ws.bins[t];
    __syncthreads();
    for (uint32_t off = 1; off < kKeyBins; off <<= 1) {
        const uint32_t o = t >= off ? s[t - off] : 0;
        __syncthreads();
        s[t] += o;
        __syncthreads();
    }
    ws.bins[t] = t ? s[t - 1] : 0;              // bucket t starts after all lower buckets
}

__global__ __launch_bounds__(kOrderBlock) void sim_order_scatter_kernel(uint32_t n_cfg, SimWs ws) {
    __shared__ uint32_t s_n[kKeyBins], s_at[kKeyBins];
    s_n[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t c = blockIdx.x * kOrderBlock + threadIdx.x;
    const uint32_t b = c < n_cfg ? ws.bucket[c] : 0u;
    uint32_t rank = 0;
    if (c < n_cfg) rank = atomicAdd(&s_n[b], 1u);
    __syncthreads();
    if (s_n[threadIdx.x]) s_at[threadIdx.x] = atomicAdd(&ws.bins[threadIdx.x], s_n[threadIdx.x]);
    __syncthreads();
    if (c < n_cfg) ws.perm[s_at[b] + rank] = c;
}

__global__ __launch_bounds__(kKeyBins) void sim_order_clear_kernel(SimWs ws) { ws.bins[threadIdx.x] = 0; }

// Heap of the decoders' finishing steps, one per lane.  The root lives in a register, node i = 1, 2, .. at position i - 1
// of the lane's LDS segment (cap positions), deeper nodes in global memory.  D-ary: the children of node i are nodes
// D i + 1 .. D i + D at positions D i .. D i + D - 1, so siblings are aligned 16-byte reads (cap is a multiple of D and at
// least D: siblings never straddle the segment's end).  Unused LDS positions hold the largest key.  (Eight children per
// node, which need fewer levels of longer comparisons, measured the same: 6.43 against 6.41 ms.)
// Key = finishing step << 10 | request; 32-bit keys when every finishing step fits 22 bits (twice the nodes in LDS).
// While the nodes of all lanes in action are in LDS, which is nearly always, the branches that look at global memory
// are left out by a choice that is uniform over the wave.
template <typename KeyT>
struct LaneHeap {
    static constexpr KeyT kEmpty = (KeyT)~(KeyT)0;
    KeyT top;             // kEmpty when there is none: above every key
    KeyT *lds;            // position j < cap
    KeyT *mem;            // position j >= cap at mem[j]
    uint32_t cap, n;
    static constexpr uint32_t D = kHeapWidth;
    struct alignas(16) Children {
        KeyT k[D];
    };
    // Waits for the global loads above it.  Where a branch that is hardly ever taken loads from global memory, the
    // wait belongs inside it: left to the value's use after the join, every lane's way there would wait for all
    // of the wave's global accesses, the stores of finishing times (a microsecond or two) among them.
    static __device__ void wait_here() { __builtin_amdgcn_s_waitcnt(0x0F70); }      // vmcnt(0)
    __device__ KeyT get(uint32_t j) const {
        KeyT k = kEmpty;
        if (j < cap) k = lds[j];
        if (j >= cap) {
            k = mem[j];
            wait_here();
        }
        return k;
    }
    __device__ void set(uint32_t j, KeyT k) {
        if (j < cap) lds[j] = k;
        if (j >= cap) mem[j] = k;
    }
    // the least of the children and which it is (keys differ)
    static __device__ KeyT least(const Children &c, uint32_t &at) {
        KeyT m = c.k[0];
#pragma unroll
        for (uint32_t j = 1; j < D; ++j) m = c.k[j] < m ? c.k[j] : m;
        at = 0;
#pragma unroll
        for (uint32_t j = 1; j < D; ++j) at = c.k[j] == m ? j : at;
        return m;
    }
    __device__ void push(KeyT key) {                // the new node rises from the end; a new least key takes the root's place
        const KeyT old = top;
        top = key < old ? key : old;
        key = key < old ? old : key;
        const uint32_t i0 = n++;                    // the new node
        if (i0 == 0) return;                        // (key is kEmpty then)
        uint32_t i = i0;
        if (__ballot(i0 > cap) == 0) {
            while (i > D) {                         // nodes 1 .. D are the root's children
                const uint32_t par = (i - 1) / D;
                const KeyT pk = lds[par - 1];
                if (pk <= key) break;
                lds[i - 1] = pk;
                i = par;
            }
            lds[i - 1] = key;
        } else {
            while (i > D) {
                const uint32_t par = (i - 1) / D;
                const KeyT pk = get(par - 1);
                if (pk <= key) break;
                set(i - 1, pk);
                i = par;
            }
            set(i - 1, key);
        }
    }
    __device__ void pop() {                         // the last node sinks from the root
        --n;
        const uint32_t end = n ? n - 1 : 0u;        // its position (with no node left: position 0, which is unused)
        uint32_t hole = 0, at;
        KeyT last;
        if (__ballot(n > cap) == 0) {
            last = lds[end];
            lds[end] = kEmpty;
            const Children k0 = *(const Children *)lds;
            KeyT best = least(k0, at);
            top = best < last ? best : last;
            if (!(best < last)) return;
            hole = at;
            for (;;) {
                const uint32_t g = D * hole + D;    // the children's positions; position end - 1 is the last in use
                const bool inside = g < end;
                const Children k = *(const Children *)(lds + (inside ? g : 0u));
                best = least(k, at);
                const bool go = inside && best < last;
                lds[hole] = go ? best : last;
                if (!go) break;
                hole = g + at;
            }
        } else {
            last = get(end);
            if (end < cap) lds[end] = kEmpty;
            const Children k0 = *(const Children *)lds;
            KeyT best = least(k0, at);
            top = best < last ? best : last;
            if (!(best < last)) return;
            hole = at;
            for (;;) {
                const uint32_t g = D * hole + D;
                if (g >= end) break;
                Children k;
                if (g < cap) k = *(const Children *)(lds + g);
                if (g >= cap) {
#pragma unroll
                    for (uint32_t j = 0; j < D; ++j) k.k[j] = g + j < end ? mem[g + j] : kEmpty;
                    wait_here();
                }
                best = least(k, at);
                if (!(best < last)) break;
                set(hole, best);
                hole = g + at;
            }
            set(hole, last);
        }
    }
};

// Pass times of one configuration with the number of layers multiplied into the layers' coefficients once.
struct LaneTimes {
    double c[N_LINEAR], m0[N_LINEAR], m1[N_LINEAR];
    double lin1, lin0;                      // norms and all-reduces: per token, per pass
    double c_lm, m0_lm, m1_lm;
    double c_att, m_att_t, m_att_k;
    double E, k;
};
__device__ inline LaneTimes lane_times(const TimeCoef &t) {
    LaneTimes r;
#pragma unroll
    for (int i = 0; i < N_LINEAR; ++i) {
        r.c[i] = t.L * t.c[i];
        r.m0[i] = t.L * t.m0[i];
        r.m1[i] = t.L * t.m1[i];
    }
    r.lin1 = t.L * fma(2.0, t.ar1, t.m_nm);
    r.lin0 = t.L * (2.0 * t.ar0);
    r.c_lm = t.c_lm; r.m0_lm = t.m0_lm; r.m1_lm = t.m1_lm;
    r.c_att = t.L * t.c_att; r.m_att_t = t.L * t.m_att_t; r.m_att_k = t.L * t.m_att_k;
    r.E = t.E; r.k = t.k;
    return r;
}
// A pass of T tokens with n_lm LM-head rows, without attention.
template <bool ADDITIVE>
__device__ inline double pass_base(const LaneTimes &t, double T, double n_lm) {
    const double eld = fmin(t.E, t.k * T);   // experts whose weights are read
    double s = fma(T, t.lin1, t.lin0);
    s += op_time<ADDITIVE>(T * t.c[OP_QKV], fma(T, t.m1[OP_QKV], t.m0[OP_QKV]));
    s += op_time<ADDITIVE>(T * t.c[OP_OPROJ], fma(T, t.m1[OP_OPROJ], t.m0[OP_OPROJ]));
    s += op_time<ADDITIVE>(T * t.c[OP_UP], fma(T, t.m1[OP_UP], eld * t.m0[OP_UP]));
    s += op_time<ADDITIVE>(T * t.c[OP_DOWN], fma(T, t.m1[OP_DOWN], eld * t.m0[OP_DOWN]));
    s += op_time<ADDITIVE>(T * t.c[OP_ROUTER], fma(T, t.m1[OP_ROUTER], t.m0[OP_ROUTER]));
    s += n_lm > 0.0 ? op_time<ADDITIVE>(n_lm * t.c_lm, fma(n_lm, t.m1_lm, t.m0_lm)) : 0.0;
    return s;
}

// The least r in 1 .. r_max with arr <= now + time_of(r), r_max when there is none; time_of grows with r.
// guess: a first estimate.  An estimate that is right or one off takes two evaluations, any other a bisection.
template <typename F>
__device__ inline uint32_t least_steps(double now, double arr, uint32_t r_max, float guess, F &&time_of) {
    uint32_t lo = 0, hi = r_max, r = guess >= 1.0f ? (guess < (float)r_max ? (uint32_t)guess : r_max) : 1u;
    bool near = true;
    while (hi - lo > 1) {
        r = r <= lo ? lo + 1 : (r >= hi ? hi - 1 : r);
        const bool reached = arr <= now + time_of((double)r);
        if (reached) hi = r; else lo = r;
        r = near ? (reached ? r - 1 : r + 1) : lo + (hi - lo) / 2;
        near = false;
    }
    return hi;
}

// What the host knows about the trace.
struct TraceSums {
    double out;             // generated tokens
    uint64_t tokens;        // prompt and generated tokens
    uint32_t longest;       // most prompt + generated tokens of one request
};

// One configuration per lane, `lanes` of them per wave (64, or fewer when there are not enough configurations for
// the chip's waves: the paths of the lanes of a wave are executed one after the other, so fewer lanes make a
// shorter instruction stream, which is what bounds the kernel: every SIMD holds one wave).
// A round of the loop does at most one of each kind of thing: one decoder leaves, one request enters, one prompt chunk is
// scheduled, a pass with prompts runs, one prompt turns into a decoder, a run of decode-only steps advances up to
// and including the step that retires the next decoder.  A lane with one event at a time takes one round per request;
// a lane with bursts takes a round per request as well, while the other lanes go on with theirs (loops over a burst
// make the whole wave wait for every lane's bursts in turn: 7000 loop turns per 1024 requests).
// CLOSED_RUNS: the run is advanced in closed form (GUIDE_SIM_CLOSED_FORM_RUNS); otherwise the clock walks through it.  A
// step's time is linear in the context while attention is bound by reading the cache at any context (nearly every
// lane), and in two pieces where it turns to arithmetic at some context, so the walk takes strides of 64 and 8 steps,
// whose times are in arithmetic progression, as long as the last step of the stride starts before the arrival that
// would end the run and lies on the same piece, and single steps after that.
// Which of the two ways a lane goes depends on its own configuration alone, never on its neighbours in the wave (which
// differ from call to call): the results of a configuration are the same bits in every list and every call.
// (The stride's sum has one rounding where 64 additions to a clock of hundreds of seconds have 64: against 80-bit
// sums the first-token times of 150 requests of up to 1500 tokens, one after the other, are 5e-15 off, step by step 7.5e-14.)
// What bounds the kernel: with one wave per SIMD a wave is a serial stream of 970 000 vector instructions (700 000 with
// closed-form runs) on average, and 40 % of its cycles are waits; the longest wave, which takes 3200 rounds, sets the time.
// 65 536 configurations x 1024 requests: 7.55 ms stepped, 5.98 ms with closed-form runs; 1999 x 97: 0.74 ms.
// Before (loops over every kind of event, two rounds per request, four predicated steps of 65 instructions at a time,
// heap segments by sequence cap, finishing times waited for by every heap read): 41.9, 13.9 and 4.1 ms.
// heap_slots: keys that the LDS behind the staged trace holds for the whole block (whole groups of siblings); they are
// shared out among the block's lanes in proportion to the most decoders each can have (its sequence cap), so that a
// lane that can run a thousand sequences gets a long segment and a lane capped at four next to nothing.
template <bool ADDITIVE, bool PREFILL_FIRST, bool CLOSED_RUNS, typename KeyT>
__global__ __launch_bounds__(kSimBlock) void simulate_kernel(GridDesc g, const DevTables *__restrict__ tab,
                                                             const TraceDev *__restrict__ trace, uint32_t n_req,
                                                             const uint32_t *__restrict__ cfg_idx,
                                                             const double *__restrict__ rate_in, uint32_t n_cfg,
                                                             guide_sim_out out, SimWs ws, TraceSums sums, uint32_t lanes,
                                                             uint32_t heap_slots, bool ordered) {
    // With 32-bit keys the whole trace is below 2^30 tokens, so blocks, budgets and steps fit 32 bits as well
    using Int = typename std::conditional<sizeof(KeyT) == 4, int32_t, long long>::type;
    constexpr Int kIntMax = sizeof(KeyT) == 4 ? (Int)0x7FFFFFFF : (Int)(1ll << 62);
    extern __shared__ __align__(16) unsigned char s_raw[];
    RequestsLds &req = *(RequestsLds *)s_raw;
    KeyT *s_heap = (KeyT *)(s_raw + sizeof(RequestsLds));
    __shared__ uint2 s_total[kSimBlock / kWave];
    for (uint32_t i = threadIdx.x; i < n_req; i += blockDim.x) {
        req.arrival[i] = trace->arrival[i];
        req.len[i] = uint2{trace->n_in[i], trace->n_out[i]};
    }
    for (uint32_t i = threadIdx.x; i < heap_slots / (16 / sizeof(KeyT)); i += blockDim.x)
        ((uint4 *)s_heap)[i] = uint4{~0u, ~0u, ~0u, ~0u};
    const uint32_t wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    // Configurations are in order of their expected concurrency, and wave w of a block takes its lanes from the
    // w-th quarter of them: lanes of a wave behave alike, and every block has waves with short and with long heaps.  The
    // last quarter, where heaps reach hundreds of keys, is dealt out lane by lane, so that no block has more of
    // the longest ones than its LDS holds (consecutive lanes there: 7.9 instead of 6.5 ms).
    const uint32_t in_part = wave & 1 ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
    const uint32_t pos = wave == kSimBlock / kWave - 1 ? (wave * lanes + lane) * gridDim.x + in_part
                                                       : (wave * gridDim.x + in_part) * lanes + lane;
    const bool in_range = lane < lanes && pos < n_cfg;
    const uint32_t c = !in_range ? 0u : ordered ? ws.perm[pos] : pos;      // the lane's configuration

    uint32_t v[kNumAxes];
    bool alive = false;                                           // this lane has a simulation to run
    uint32_t max_seqs = 1, mbt = 1;
    double rate = 1.0;
    Int n_blk = 0;
    LaneTimes lt;
    Div32 dblk = make_div32(1);
    // KV blocks of a request of `tok` >= 1 tokens: ceil(tok / blk) without the 32-bit overflow of tok + blk - 1
    auto blocks_of = [&](uint32_t tok) { return (Int)div32(tok - 1, dblk) + 1; };
    if (in_range) {
        const bool bad_index = decode_sim_index(tab->axis_vals, g, cfg_idx[c], v);
        max_seqs = v[AX_BATCH]; mbt = v[AX_MBT];
        const guide_hw hw = tab->hw[v[AX_HW]];
        rate = rate_in[c];
        const Coef cf = make_coef(tab->models[v[AX_MODEL]], v[AX_TP], v[AX_WBITS]);
        lt = lane_times(make_time_coef(cf, 1.0 / hw.peak_flops, 1.0 / hw.hbm_bw, 1.0 / hw.link_bw, hw.link_lat));
        dblk = make_div32(v[AX_BLK]);
        // KV pool in blocks; every request must fit on its own
        const double c_avail = hw.cap_bytes - cf.w_gpu;
        if (c_avail > 0.0) {
            const double nb = floor(c_avail / ((double)v[AX_BLK] * cf.kv_tok));
            n_blk = nb >= (double)kIntMax ? kIntMax : (Int)nb;
        }
        if (bad_index || !(c_avail > 0.0) || blocks_of(sums.longest) > n_blk || !(rate > 0.0)) {
            out.ttft_p50[c] = INFINITY; out.ttft_p99[c] = INFINITY; out.mean_tpot[c] = INFINITY; out.tokens_s[c] = 0.0;
            out.status[c] = (bad_index || !(rate > 0.0)) ? GUIDE_SIM_BAD_INPUT : GUIDE_SIM_INFEASIBLE;
            out.n_steps[c] = 0; out.n_request_steps[c] = 0;
        } else {
            alive = true;
        }
    }

    // LDS segments of the heaps: a lane can have at most min(sequence cap, requests) decoders, one of them in a
    // register; when the block's lanes want more than the LDS holds, every segment shrinks by the same factor
    LaneHeap<KeyT> heap;
    {
        const uint32_t most = max_seqs < n_req ? max_seqs : n_req;
        // most - 1 positions at most, and not many more than the pool holds requests of average length; three times
        // the expected concurrency first, what is left over in proportion to the rest
        const float mean_blocks = (float)sums.tokens / (float)n_req / (float)dblk.d + 0.5f;
        const float pool = fminf(1.5f * (float)n_blk / mean_blocks + 4.0f, 2048.0f);
        auto groups = [](uint32_t x) { return (x + kHeapWidth - 1) / kHeapWidth * kHeapWidth; };
        const uint32_t bound = groups((most < (uint32_t)pool ? most : (uint32_t)pool) - 1u);
        const uint32_t likely = ordered ? groups((uint32_t)(3.0f * expected_of(alive ? ws.bucket[c] : 0u)) + 16u) : bound;
        const uint32_t full = alive ? (bound < kHeapWidth ? kHeapWidth : bound) : 0u, want = alive && likely < full ? likely : full;
        const uint32_t wave_want = wave_sum(want), wave_full = wave_sum(full);
        if (lane == 0) s_total[wave] = uint2{wave_want, wave_full};
        __syncthreads();                                // the trace and the empty heaps are staged as well
        uint32_t total = 0, total_full = 0;
        for (uint32_t w = 0; w < kSimBlock / kWave; ++w) {
            total += s_total[w].x;
            total_full += s_total[w].y;
        }
        // (heap_slots is at least a group per thread whenever the wants do not fit, so every lane in use keeps one)
        uint32_t cap = want;
        if (total > heap_slots)
            cap = kHeapWidth + (uint32_t)((double)(want - kHeapWidth) * ((double)(heap_slots - kHeapWidth * kSimBlock) / (double)total)) /
                                   kHeapWidth * kHeapWidth;
        else if (total_full > total)
            cap = want + (uint32_t)((double)(full - want) * fmin((double)(heap_slots - total) / (double)(total_full - total), 1.0)) /
                             kHeapWidth * kHeapWidth;
        if (!alive) cap = 0;
        const uint32_t incl = wave_scan_sum(cap);
        __syncthreads();
        if (lane == kWave - 1) s_total[wave].x = incl;
        __syncthreads();
        uint32_t off = incl - cap;
        for (uint32_t w = 0; w < wave; ++w) off += s_total[w].x;
        heap.lds = s_heap + off;
        heap.cap = cap;
    }
    // attention bound by reading the cache at every context: step times are linear (in every lane: wave_linear, which only
    // leaves work out that changes nothing in such a lane)
    const bool lane_linear = ADDITIVE || lt.c_att <= lt.m_att_k;
    const bool wave_linear = ADDITIVE || __ballot(alive && !lane_linear) == 0;
    if (!alive) return;

    heap.top = LaneHeap<KeyT>::kEmpty;
    heap.mem = (KeyT *)(ws.heap + (size_t)pos * n_req);
    heap.n = 0;
    double *first = ws.first + (size_t)c * n_req, *fin = ws.fin + (size_t)c * n_req;

    // arrival / rate: the reciprocal's product with one correction step rounds as the division does, unless the quotient lies
    // within 2^-50 units of its last place of a rounding boundary; rates and traces at the ends of the range are divided
    const double last_arrival = req.arrival[n_req - 1];
    const bool plain_rate = rate >= 0x1p-400 && rate <= 0x1p400 && last_arrival <= 0x1p400;
    const bool wave_plain = __ballot(!plain_rate) == 0;
    const double r_rate = 1.0 / rate;
    auto arrival_of = [&](double a) {
        const double q = a * r_rate;
        double t = fma(fma(-q, rate, a), r_rate, q);
        if (!wave_plain) {
            asm volatile("");                           // keeps the division out of the other lanes' way
            t = plain_rate ? t : a / rate;
        }
        return t;
    };
    const Int budget_full = (uint64_t)mbt > (uint64_t)(kIntMax / 2) ? kIntMax / 2 : (Int)mbt;   // beyond every trace

    double now = 0.0, max_fin = -INFINITY, s_ctx = 0.0;     // s_ctx: total context, an integer far below 2^53
    // prompts [comp, next) are admitted and have not emitted their first token; the next one to schedule is h, of which
    // `done` tokens have been computed; pend: prompts from comp on whose last chunk was in the pass just run
    uint32_t next = 0, comp = 0, h = 0, done = 0, pend = 0, n_dec = 0, n_done = 0;
    double c_T = 0.0, c_Q = 0.0, c_K = 0.0;                 // chunks scheduled for the next pass: tokens, workload, context
    uint32_t chunks = 0, n_full = 0;                        // their number, and prompts that they complete
    Int used = 0;                                           // their tokens
    uint64_t step = 0, n_rs = 0;
    KeyT dstep = 0;                                         // steps in which decoders ran
    Int free_blk = n_blk;
    uint32_t status = GUIDE_SIM_OK;
    const uint64_t step_bound = (uint64_t)n_req + sums.tokens;      // every step consumes at least one token of some request
    const uint32_t last_req = n_req - 1;
    auto at_most = [&](uint32_t r) { return r < last_req ? r : last_req; };
    double arr_next = arrival_of(req.arrival[0]);           // arrival time of request `next`
    Int need_next = blocks_of(req.len[0].x + req.len[0].y);
    double kept_base = 0.0;                                 // pass_base of kept_dec decode tokens
    uint32_t kept_dec = 0;

    for (;;) {
        // everything that the steps below read from LDS, requested together
        const uint2 l_h = req.len[at_most(h)], l_comp = req.len[at_most(comp)], l_next = req.len[at_most(next + 1)];
        const double a_next = req.arrival[at_most(next + 1)];
        bool moved = false;
        // 1. a decoder that has emitted its last token leaves (an empty heap's top is beyond every step)
        if ((heap.top >> 10) == dstep) {
            const uint32_t r = (uint32_t)(heap.top & 1023u);
            const uint2 len = req.len[r];
            heap.pop();
            free_blk += blocks_of(len.x + len.y);
            --n_dec;
            s_ctx -= (double)(len.x + len.y);
            ++n_done;
            fin[r] = now;
            max_fin = now;
            moved = true;
        }
        if (n_done == n_req) break;
        // 2. idle: jump to the next arrival
        const uint32_t n_active = (next - comp) + n_dec;
        if (n_active == 0 && next < n_req) now = arr_next > now ? arr_next : now;
        // 3. FCFS admission of one request, if it can enter.  (Decoders that still have to leave, or prompts that turn into
        // decoders, only make room: whoever enters before would enter after.)
        auto admissible = [&](uint32_t active) {
            return next < n_req && active < max_seqs && arr_next <= now && need_next <= free_blk;
        };
        if (admissible(n_active)) {
            free_blk -= need_next;
            ++next;
            arr_next = next < n_req ? arrival_of(a_next) : INFINITY;
            need_next = blocks_of(l_next.x + l_next.y);
            moved = true;
        }
        const bool leaving = (heap.top >> 10) == dstep;
        // 4. schedule one prompt chunk.  Split-fuse: the budget that the decoders leave, whose number is final once nobody
        // leaves or joins any more; a whole prompt may go in before when it fits for sure.  Prefill-first:
        // whole prompts, as many as fit the budget, the first always.
        {
            const Int rem = (Int)(l_h.x - done);
            const Int left = PREFILL_FIRST ? budget_full - used : budget_full - (Int)(n_dec + pend) - used;
            const bool fits = PREFILL_FIRST ? (chunks == 0 || rem <= left)
                                            : (rem <= left || (left > 0 && !leaving && pend == 0));
            if (h < next && fits) {
                const Int ch = PREFILL_FIRST ? rem : (rem < left ? rem : left);
                used += ch;
                done += (uint32_t)ch;
                const double C = (double)ch, ctx = (double)done;
                c_T += C;
                c_Q = fma(C, ctx, c_Q);
                c_K += ctx;
                ++chunks;
                if (ch == rem) {
                    ++n_full;
                    ++h;
                    done = 0;
                }
                moved = true;
            }
        }
        // 5. a pass with prompts, once nothing is left to be done before it: one token per decoder (prefill-first:
        // the decoders pause) and the scheduled chunks
        const bool settled = !leaving && pend == 0 && !admissible((next - comp) + n_dec);
        if (settled && comp < next) {
            const bool more = h < next && (PREFILL_FIRST ? (Int)(req.len[at_most(h)].x) <= budget_full - used
                                                         : budget_full - (Int)n_dec - used > 0);
            if (!more) {
                const double d = PREFILL_FIRST ? 0.0 : (double)n_dec, ctx = PREFILL_FIRST ? 0.0 : s_ctx;
                const double T = c_T + d, Q = c_Q + ctx, K = c_K + ctx;
                now += pass_base<ADDITIVE>(lt, T, d + (double)n_full) +
                       op_time<ADDITIVE>(Q * lt.c_att, fma(K, lt.m_att_k, T * lt.m_att_t));
                ++step;
                n_rs += chunks;
                if (!PREFILL_FIRST) {
                    n_rs += n_dec;
                    if (n_dec > 0) ++dstep;
                    s_ctx += d;
                }
                pend = n_full;
                c_T = c_Q = c_K = 0.0;
                chunks = n_full = 0;
                used = 0;
                moved = true;
            }
        }
        // 6. a prompt completed in the last pass emits its first token
        if (pend > 0) {
            const uint32_t r = comp;
            first[r] = now;
            if (l_comp.y == 1) {
                free_blk += blocks_of(l_comp.x + 1);
                ++n_done;
                fin[r] = now;
                max_fin = now;
            } else {
                ++n_dec;
                s_ctx += (double)(l_comp.x + 1);
                heap.push((KeyT)(((dstep + (KeyT)(l_comp.y - 1)) << 10) | r));
            }
            ++comp;
            --pend;
            moved = true;
        }
        // 7. run of decode-only steps: no prompt is waiting, and nothing changes until the first decoder emits its
        // last token or a request that could be admitted arrives.
        if (comp == next && n_dec > 0 && (heap.top >> 10) != dstep) {
            const double T = (double)n_dec;
            if (kept_dec != n_dec) {
                kept_base = pass_base<ADDITIVE>(lt, T, T);
                kept_dec = n_dec;
            }
            const bool can_admit = next < n_req && n_dec < max_seqs && need_next <= free_blk;
            const double arr_stop = can_admit ? arr_next : __builtin_nan("");      // compares false: nothing ends the run early
            const uint32_t total = (uint32_t)((heap.top >> 10) - dstep);  // steps up to the one that retires a decoder
            // time of a step at context c: base + max(c_att c, m_att_k c + T m_att_t)
            const double base = kept_base, base_m = fma(T, lt.m_att_t, base);
            const double slope = ADDITIVE ? lt.c_att + lt.m_att_k : lt.m_att_k;
            auto step_time = [&](double ctx) {
                const double tm = fma(ctx, slope, base_m);
                return wave_linear ? tm : fmax(fma(ctx, lt.c_att, base), tm);      // (tm is the larger in a linear lane)
            };
            uint32_t run = 0;
            if (CLOSED_RUNS) {
                // all steps before the retiring one, or the least number after which the arrival has come
                const uint32_t r_max = total - 1;
                if (r_max > 0 && !(arr_stop <= now)) {
                    const double h_T = 0.5 * T;
                    float guess = 1.0f;
                    if (can_admit) {
                        // time(r) = p r + q r^2 up to rounding on the side that the run starts on; its root in single
                        // precision is the first guess
                        const double rem = arr_stop - now;
                        const bool arith = !lane_linear && fma(s_ctx, lt.c_att, base) >= fma(s_ctx, slope, base_m);
                        const double sl = arith ? lt.c_att : slope;
                        const float q = (float)(sl * h_T), p = (float)fma(sl, s_ctx - h_T, arith ? base : base_m), rf = (float)rem;
                        guess = ceilf(2.0f * rf * __builtin_amdgcn_rcpf(p + __builtin_amdgcn_sqrtf(fmaf(p, p, 4.0f * q * rf))));
                    }
                    auto advance = [&](auto &&time_of) {
                        run = can_admit ? least_steps(now, arr_stop, r_max, guess, time_of) : r_max;
                        now += time_of((double)run);
                    };
                    if (lane_linear)
                        advance([&](double r) { return r * fma(slope, fma(h_T, r - 1.0, s_ctx), base_m); });
                    else
                        advance([&](double r) {
                            return fma(r, base, attention_series<ADDITIVE>(lt.c_att, lt.m_att_k, T * lt.m_att_t, s_ctx - T, T,
                                                                           fast_recip(T), r));
                        });
                }
                if (run == r_max && !(arr_stop <= now)) {
                    now += step_time(fma((double)run, T, s_ctx));
                    ++run;
                }
            } else if (lane_linear) {
                const double dt = slope * T;
                double t0 = fma(s_ctx, slope, base_m);
                // strides of 64, then of 8 steps, whose times are in arithmetic progression, while the last step
                // of the stride would still start before the arrival; then step by step
                auto stride = [&](auto steps) {
                    constexpr double kS = decltype(steps)::value;
                    while (run + (uint32_t)kS <= total) {
                        const double to_last = now + fma(0.5 * (kS - 1.0) * (kS - 2.0), dt, (kS - 1.0) * t0);
                        if (arr_stop <= to_last) break;
                        now += fma(0.5 * kS * (kS - 1.0), dt, kS * t0);
                        t0 = fma(kS, dt, t0);
                        run += (uint32_t)kS;
                    }
                };
                stride(std::integral_constant<int, 64>{});
                t0 = fma(fma((double)run, T, s_ctx), slope, base_m);
                stride(std::integral_constant<int, 8>{});
                t0 = fma(fma((double)run, T, s_ctx), slope, base_m);
                bool go = true;
#pragma unroll
                for (int j = 0; j < 7; ++j) {
                    go = go && run < total && !(arr_stop <= now);
                    const double n = now + fma((double)j, dt, t0);
                    now = go ? n : now;
                    run += go ? 1u : 0u;
                }
            } else {
                // Attention may turn from read bound to bound by arithmetic at some context, and stays so (its slope is
                // the greater one): strides whose first and last step lie on the same side, as above; those that
                // do not are left to shorter ones and to single steps, after which the next round goes on.
                auto stride = [&](auto steps) {
                    constexpr double kS = decltype(steps)::value;
                    while (run + (uint32_t)kS <= total) {
                        const double ctx = fma((double)run, T, s_ctx), last = fma(kS - 1.0, T, ctx);
                        const double t_c = fma(ctx, lt.c_att, base), t_m = fma(ctx, slope, base_m);
                        const bool arith = t_c >= t_m;
                        if (!arith && fma(last, lt.c_att, base) > fma(last, slope, base_m)) break;
                        const double t0 = arith ? t_c : t_m, dt = (arith ? lt.c_att : slope) * T;
                        const double to_last = now + fma(0.5 * (kS - 1.0) * (kS - 2.0), dt, (kS - 1.0) * t0);
                        if (arr_stop <= to_last) break;
                        now += fma(0.5 * kS * (kS - 1.0), dt, kS * t0);
                        run += (uint32_t)kS;
                    }
                };
                stride(std::integral_constant<int, 64>{});
                stride(std::integral_constant<int, 8>{});
                bool go = true;
#pragma unroll
                for (int j = 0; j < 7; ++j) {
                    go = go && run < total && !(arr_stop <= now);
                    const double n = now + step_time(fma((double)run, T, s_ctx));
                    now = go ? n : now;
                    run += go ? 1u : 0u;
                }
            }
            step += run;
            dstep += (KeyT)run;
            n_rs += (uint64_t)run * n_dec;
            s_ctx = fma((double)run, T, s_ctx);
            moved = moved || run > 0;
        }
        if (step > step_bound || !moved) {                  // a round always moves something
            status = GUIDE_SIM_INTERNAL;
            break;
        }
    }

    out.tokens_s[c] = status == GUIDE_SIM_OK ? sums.out / (max_fin - req.arrival[0] / rate) : 0.0;
    out.status[c] = status;
    out.n_steps[c] = step;
    out.n_request_steps[c] = n_rs;
    if (status != GUIDE_SIM_OK) {
        out.ttft_p50[c] = INFINITY; out.ttft_p99[c] = INFINITY; out.mean_tpot[c] = INFINITY;
    }
}

// One wave per simulated configuration that ended normally.  TTFT of request i = first token time - arrival /
// rate; the 1024 values (absent requests count as +inf) are sorted inside the wave's registers, 16 per lane, by
// a bitonic network in which every compare-exchange puts the smaller value at the smaller index: element
// e = 16 * lane + register; a stage pairs e with e ^ m, which is another register of the same lane while m < 16
// and the same-numbered (or mirrored) register of lane ^ (m / 16) otherwise.  Then nearest-rank
// p50 = sorted[ceil(n/2) - 1] and p99 = sorted[ceil(0.99 n) - 1]; mean TPOT = mean over requests with more than
// one token of (finish - first token) / (tokens - 1).
constexpr uint32_t kPerLane = GUIDE_MAX_REQUESTS / kWave;       // 16
static_assert(kPerLane == 16, "the network below is written for 16 values per lane");

constexpr uint32_t top_bit(uint32_t x) { return x < 2 ? x : 2 * top_bit(x / 2); }
// compare-exchange inside a lane: the smaller value to the smaller register
__device__ inline void cx(double &a, double &b) {
    const double lo = fmin(a, b), hi = fmax(a, b);
    a = lo;
    b = hi;
}
// One stage of the network.  MASK: the xor mask on element numbers.
template <uint32_t MASK>
__device__ inline void sort_stage(double (&v)[kPerLane], uint32_t lane) {
    if constexpr (MASK < kPerLane) {
#pragma unroll
        for (uint32_t r = 0; r < kPerLane; ++r)
            if ((r ^ MASK) > r) cx(v[r], v[r ^ MASK]);
    } else {
        constexpr uint32_t kLaneMask = MASK / kPerLane, kRegMask = MASK % kPerLane;     // kRegMask: 0 or 15 (mirror)
        // this lane holds the smaller indices of its pairs when the top bit of the lane mask is clear in its number
        constexpr uint32_t kTop = top_bit(kLaneMask);
        const bool keep_min = (lane & kTop) == 0;
        double o[kPerLane];
#pragma unroll
        for (uint32_t r = 0; r < kPerLane; ++r) o[r] = __shfl_xor(v[r ^ kRegMask], (int)kLaneMask, kWave);
#pragma unroll
        for (uint32_t r = 0; r < kPerLane; ++r) v[r] = keep_min ? fmin(v[r], o[r]) : fmax(v[r], o[r]);
    }
}
// Merge of sorted runs of K / 2 elements into sorted runs of K: the mirror stage, then halving distances.
template <uint32_t K>
__device__ inline void sort_merge(double (&v)[kPerLane], uint32_t lane) {
    sort_stage<K - 1>(v, lane);
    if constexpr (K >= 4) sort_stage<K / 4>(v, lane);
    if constexpr (K >= 8) sort_stage<K / 8>(v, lane);
    if constexpr (K >= 16) sort_stage<K / 16>(v, lane);
    if constexpr (K >= 32) sort_stage<K / 32>(v, lane);
    if constexpr (K >= 64) sort_stage<K / 64>(v, lane);
    if constexpr (K >= 128) sort_stage<K / 128>(v, lane);
    if constexpr (K >= 256) sort_stage<K / 256>(v, lane);
    if constexpr (K >= 512) sort_stage<K / 512>(v, lane);
    if constexpr (K >= 1024) sort_stage<K / 1024>(v, lane);
}
// element `e` of the sorted sequence, in every lane
__device__ inline double sorted_at(const double (&v)[kPerLane], uint32_t e) {
    double x = v[0];
#pragma unroll
    for (uint32_t r = 1; r < kPerLane; ++r) x = (e % kPerLane) == r ? v[r] : x;
    return __shfl(x, (int)(e / kPerLane), kWave);
}

__global__ __launch_bounds__(kPctBlock) void percentile_kernel(SimWs ws, const TraceDev *__restrict__ trace,
                                                               const double *__restrict__ rate_in, uint32_t n_req,
                                                               uint32_t n_cfg, guide_sim_out out) {
    const uint32_t lane = threadIdx.x % kWave;
    const uint32_t c = blockIdx.x * (kPctBlock / kWave) + threadIdx.x / kWave;      // wave-uniform
    if (c >= n_cfg || out.status[c] != GUIDE_SIM_OK) return;
    const double rate = rate_in[c];
    const double *first = ws.first + (size_t)c * n_req, *fin = ws.fin + (size_t)c * n_req;
    double v[kPerLane];
    double tp = 0.0;
    uint32_t n_tp = 0;
#pragma unroll
    for (uint32_t r = 0; r < kPerLane; ++r) {
        const uint32_t i = r * kWave + lane;                // coalesced; the sort does not care where a value starts
        double t = INFINITY;
        if (i < n_req) {
            const double f = first[i];
            t = f - trace->arrival[i] / rate;
            const uint32_t n_out = trace->n_out[i];
            if (n_out > 1) {
                tp += (fin[i] - f) / (double)(n_out - 1);
                ++n_tp;
            }
        }
        v[r] = t;
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        tp += __shfl_xor(tp, off, kWave);
        n_tp += __shfl_xor(n_tp, off, kWave);
    }
    sort_merge<2>(v, lane);
    sort_merge<4>(v, lane);
    sort_merge<8>(v, lane);
    sort_merge<16>(v, lane);
    sort_merge<32>(v, lane);
    sort_merge<64>(v, lane);
    sort_merge<128>(v, lane);
    sort_merge<256>(v, lane);
    sort_merge<512>(v, lane);
    sort_merge<1024>(v, lane);
    const double p50 = sorted_at(v, (n_req + 1) / 2 - 1);
    const double p99 = sorted_at(v, (uint32_t)((99ull * n_req + 99) / 100 - 1));
    if (lane == 0) {
        out.ttft_p50[c] = p50;
        out.ttft_p99[c] = p99;
        out.mean_tpot[c] = n_tp ? tp / (double)n_tp : 0.0;
    }
}

}  // namespace

size_t simulate_workspace_bytes(uint32_t n_cfg, uint32_t n_req) {
    return (size_t)n_cfg * n_req * 24 + (size_t)n_cfg * 8 + kKeyBins * 4 + 256;
}

hipError_t launch_simulate(const GridDesc &g, const DevTables *tab, const TraceDev *trace, uint32_t n_req,
                           const uint32_t *cfg_idx, const double *rate, uint32_t n_cfg, bool additive,
                           bool prefill_first, bool closed_runs, const guide_sim_out &out, void *ws_, hipStream_t stream,
                           double sum_in, double sum_out, uint32_t longest) {
    const SimWs ws = sim_ws(ws_, n_cfg, n_req);
    const TraceSums sums{sum_out, (uint64_t)(sum_in + sum_out), longest};
    // Lanes in use per wave: 64 once the configurations fill a wave per SIMD, otherwise as few as still give every
    // SIMD at most one wave.
    const uint32_t simds = device_cus() * 4;
    uint32_t lanes = kWave;
    while (lanes > 1 && (uint64_t)n_cfg <= (uint64_t)(lanes / 2) * simds) lanes /= 2;
    const uint32_t per_block = kSimBlock / kWave * lanes;
    // LDS beyond the staged trace holds heap nodes of the block's lanes; 32-bit keys when every finishing step
    // (at most the trace's generated tokens) fits 22 bits and the trace's tokens fit 30
    const bool key32 = sum_out < 4194303.0 && sum_in < 1073700000.0;
    const size_t key_bytes = key32 ? sizeof(uint32_t) : sizeof(uint64_t);
    int dev = 0, lds_max = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return e;
    const size_t staged = sizeof(RequestsLds), fixed = staged + kSimStaticLds;
    if ((size_t)lds_max < fixed + kSimBlock * kHeapWidth * key_bytes) return hipErrorInvalidValue;
    size_t heap_bytes = (size_t)lds_max - fixed;
    const size_t most = (size_t)per_block * (n_req + 2 * kHeapWidth) * key_bytes;      // no lane needs more
    heap_bytes = heap_bytes < most ? heap_bytes : most;
    heap_bytes -= heap_bytes % (kHeapWidth * sizeof(uint64_t));
    const uint32_t heap_slots = (uint32_t)(heap_bytes / key_bytes);
    const size_t lds_bytes = staged + heap_bytes;
    const dim3 grid((n_cfg + per_block - 1) / per_block), block(kSimBlock);
    const dim3 ogrid((n_cfg + kOrderBlock - 1) / kOrderBlock), oblock(kOrderBlock);
    const bool ordered = lanes > 1 && n_req >= kOrderRequests;      // (otherwise every lane's heap fits the LDS)
    if (ordered) {
        hipLaunchKernelGGL(sim_order_clear_kernel, dim3(1), dim3(kKeyBins), 0, stream, ws);
        if (additive)
            hipLaunchKernelGGL(sim_order_count_kernel<true>, ogrid, oblock, 0, stream, g, tab, n_req, cfg_idx, rate, n_cfg, ws, sum_in, sum_out);
        else
            hipLaunchKernelGGL(sim_order_count_kernel<false>, ogrid, oblock, 0, stream, g, tab, n_req, cfg_idx, rate, n_cfg, ws, sum_in, sum_out);
        hipLaunchKernelGGL(sim_order_scan_kernel, dim3(1), dim3(kKeyBins), 0, stream, ws);
        hipLaunchKernelGGL(sim_order_scatter_kernel, ogrid, oblock, 0, stream, n_cfg, ws);
    }
    const int variant = (additive ? 8 : 0) | (prefill_first ? 4 : 0) | (closed_runs ? 2 : 0) | (key32 ? 1 : 0);
#define GUIDE_SIM(A, P, C, K32)                                                                                    \
    case ((A ? 8 : 0) | (P ? 4 : 0) | (C ? 2 : 0) | (K32 ? 1 : 0)): {                                               \
        auto kern = simulate_kernel<A, P, C, std::conditional<K32, uint32_t, uint64_t>::type>;                      \
        e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);    \
        if (e != hipSuccess) return e;                                                                              \
        hipLaunchKernelGGL(kern, grid, block, lds_bytes, stream, g, tab, trace, n_req, cfg_idx, rate, n_cfg, out, ws, \
                           sums, lanes, heap_slots, ordered);                                                               \
        break;                                                                                                      \
    }
    switch (variant) {
        GUIDE_SIM(false, false, false, false) GUIDE_SIM(false, false, false, true) GUIDE_SIM(false, false, true, false)
        GUIDE_SIM(false, false, true, true) GUIDE_SIM(false, true, false, false) GUIDE_SIM(false, true, false, true)
        GUIDE_SIM(false, true, true, false) GUIDE_SIM(false, true, true, true) GUIDE_SIM(true, false, false, false)
        GUIDE_SIM(true, false, false, true) GUIDE_SIM(true, false, true, false) GUIDE_SIM(true, false, true, true)
        GUIDE_SIM(true, true, false, false) GUIDE_SIM(true, true, false, true) GUIDE_SIM(true, true, true, false)
        GUIDE_SIM(true, true, true, true)
    }
#undef GUIDE_SIM
    hipLaunchKernelGGL(percentile_kernel, dim3((n_cfg + kPctBlock / kWave - 1) / (kPctBlock / kWave)), dim3(kPctBlock), 0,
                       stream, ws, trace, rate, n_req, n_cfg, out);
    return hipGetLastError();
}

}  // namespace guide
