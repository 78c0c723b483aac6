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
//     per-lane queue keyed by finishing step, in LDS as far as it goes, and
//     their number and total context are two running numbers.
// A request therefore costs a few pass-time evaluations, a push and a pop;
// the steps in between are advanced at once.
#include <type_traits>

#include "kernels.hpp"
#include "perf_model.hpp"
#include "reduce.hpp"

namespace guide {

namespace {

constexpr uint32_t kSimWaves = 8;        // most waves of a block; a block stages the trace once, the rest of its LDS holds queues
constexpr uint32_t kSimBlock = kSimWaves * kWave;
constexpr uint32_t kPctBlock = 256;
constexpr size_t kSimStaticLds = 128;    // the simulation kernel's own static LDS (wave totals)

// A request as the simulation kernel keeps it in LDS; two entries past the last one stand for `none left` (arrival: no
// number, which compares false with everything).
struct alignas(16) Request {
    double arrival;              // at unit rate
    uint32_t in, out;            // prompt and generated tokens
};
struct RequestsLds {
    Request r[GUIDE_MAX_REQUESTS + 2];
};

constexpr uint32_t kHeapWidth = 4;     // children per heap node
constexpr uint32_t kKeyBins = 1024;      // buckets of the expected-concurrency ordering
// Lists are ordered where that saves more than its four launches (17 us): when lanes share a wave at all, and blocks of several
// waves from 64 requests on, blocks of one wave when LDS does not hold a slot for every request (353 requests).  Ordered / as
// given, in us: 5000 x 16 83 / 64, 5000 x 64 248 / 231, 5000 x 352 1300 / 1286; 65 536 x 16 114 / 98, 65 536 x 64 277 / 272,
// 65 536 x 128 535 / 551; 40 000 x 64 270 / 269, 40 000 x 96 407 / 414; 200 000 x 48 754 / 758, 200 000 x 64 945 / 955.
constexpr uint32_t kOrderRequests = 64;

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
                                                                      SimWs ws, double sum_in, double sum_out,
                                                                      double unit_rate) {
    __shared__ uint32_t s_n[kKeyBins];
    s_n[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t c = blockIdx.x * kOrderBlock + threadIdx.x;
    if (c < n_cfg) {
        uint32_t v[kNumAxes];
        const bool bad = decode_sim_index(tab->axis_vals, g, cfg_idx[c], v);
        uint32_t b = 0;
        const double rate = rate_in[c] * unit_rate;                 // requests per second
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
// least D: siblings never straddle the segment's end).  Unused LDS positions hold the largest key.
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

// A lane's keys that found no room in LDS: a 4-ary min-heap in global memory, its root in a register; the children of node i
// are nodes D i + 1 .. D i + D, node j at mem[j - 1].
struct MemHeap {
    static constexpr uint32_t kEmpty = ~0u, D = kHeapWidth;
    uint32_t top, *mem, n;
    __device__ void push(uint32_t key) {
        const uint32_t old = top;
        top = key < old ? key : old;
        key = key < old ? old : key;
        uint32_t i = n++;
        if (i == 0) return;                             // (key is kEmpty then)
        while (i > D) {
            const uint32_t par = (i - 1) / D, pk = mem[par - 1];
            LaneHeap<uint32_t>::wait_here();
            if (pk <= key) break;
            mem[i - 1] = pk;
            i = par;
        }
        mem[i - 1] = key;
    }
    __device__ void pop() {                             // the last node sinks from the root
        top = kEmpty;
        if (--n == 0) return;
        const uint32_t end = n - 1, last = mem[end];    // positions 0 .. end - 1 are left
        top = last;
        uint32_t hole = ~0u;                            // the root
        for (uint32_t g = 0; g < end;) {
            uint32_t k[D], at = 0, best;
#pragma unroll
            for (uint32_t j = 0; j < D; ++j) k[j] = g + j < end ? mem[g + j] : kEmpty;
            LaneHeap<uint32_t>::wait_here();
            best = k[0];
#pragma unroll
            for (uint32_t j = 1; j < D; ++j) best = k[j] < best ? k[j] : best;
#pragma unroll
            for (uint32_t j = 1; j < D; ++j) at = k[j] == best ? j : at;       // (keys differ; 0 when none of the others is it)
            if (!(best < last)) break;
            if (hole == ~0u) top = best; else mem[hole] = best;
            hole = g + at;
            g = D * hole + D;
        }
        if (hole != ~0u) mem[hole] = last;
    }
};

// The decoders of a lane by finishing step when keys have 32 bits.  Keys (step << 10 | slot) lie in slots of the lane's LDS
// segment in any order, sixteen to a block; the least key of every block is kept beside them, the least of all in a
// register, and the request of a slot in a table of its own.  A push is two stores and a minimum that nothing waits for;
// a pop reads the sixteen keys of the block it leaves a hole in and the least keys of the blocks around it, all at once, and
// takes minima (with more than sixteen blocks, their least keys by sixteens make a third level): an LDS latency or two and no
// loop, whatever the lane's neighbours do: 700 - 950 cycles a round with the retirement, the push 350 (a 4-ary heap: a latency
// per level, and every lane waited for the deepest: 700 - 1570 and 430 - 730).  Free slots form a list through the request table.
// Decoders beyond the segment go to a heap in global memory (MemHeap).
// Segment: keys[cap], then the blocks' least keys (a multiple of four of them), then those of sixteen blocks each (none or
// four), then the requests (16 bits each); cap is a multiple of 16, and 0 only in lanes that have nothing to simulate.
struct SlotQueue {
    static constexpr uint32_t kEmpty = ~0u, kPer = 16, kNoSlot = 0xFFFFu;
    // LDS bytes of n blocks, and what each block after the first takes at most beside the first one's
    static constexpr uint32_t kFirstBytes = kPer * 6 + 16, kMoreBytes = kPer * 6 + 5;
    static __host__ __device__ uint32_t bytes(uint32_t n) { return n * kPer * 6 + (n + 3) / 4 * 16 + (n > kPer ? 16u : 0u); }
    static_assert(GUIDE_MAX_REQUESTS <= 4 * kPer * kPer, "four superblocks");
    uint32_t top;                     // kEmpty when there is none: above every key
    uint32_t keys, low, req;          // byte offsets of the segment's parts
    uint32_t cap, used, free_;        // slots; slots ever taken; first of the list of free slots below `used`
    uint32_t last_group;              // byte offset of the last group of four blocks' least keys
    uint32_t super_;                  // ... of the least keys of sixteen blocks each; 0: no more than sixteen blocks
    MemHeap over;                     // the decoders that found no slot: keys step << 10 | request
    __device__ void init(uint32_t offset, uint32_t blocks, uint32_t *mem) {
        top = kEmpty;
        cap = blocks * kPer;
        keys = offset;
        low = keys + cap * 4;
        const uint32_t groups = (blocks + 3) / 4;
        last_group = low + (groups - 1) * 16;
        super_ = blocks > kPer ? low + groups * 16 : 0u;
        req = low + groups * 16 + (blocks > kPer ? 16u : 0u);
        used = 0;
        free_ = kNoSlot;
        over = MemHeap{kEmpty, mem, 0};
    }
    __device__ uint32_t due() const { return (top < over.top ? top : over.top) >> 10; }
    template <typename T>
    static __device__ T &at(unsigned char *lds, uint32_t offset) { return *(T *)(lds + offset); }
    // The request of the least key in a slot (anything when there is none).
    __device__ uint32_t first_request(unsigned char *lds) const {
        return at<uint16_t>(lds, req + (top == kEmpty ? 0u : (top & 1023u) * 2));
    }
    // supers: some lane of the wave has more than sixteen blocks (uniform).
    __device__ void put(unsigned char *lds, uint32_t step, uint32_t r, bool supers) {
        const bool reuse = free_ != kNoSlot;
        const uint32_t slot = reuse ? free_ : used;
        auto store = [&]() {
            const uint32_t next = at<uint16_t>(lds, req + slot * 2), key = step << 10 | slot;
            asm volatile("" ::: "memory");              // a wave's LDS operations are done in program order
            at<uint32_t>(lds, keys + slot * 4) = key;
            at<uint16_t>(lds, req + slot * 2) = (uint16_t)r;
            __hip_atomic_fetch_min(&at<uint32_t>(lds, low + slot / kPer * 4), key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            if (supers && super_)
                __hip_atomic_fetch_min(&at<uint32_t>(lds, super_ + slot / (kPer * kPer) * 4), key, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WAVEFRONT);
            free_ = reuse ? next : kNoSlot;
            used += reuse ? 0u : 1u;
            top = key < top ? key : top;
        };
        if (__ballot(slot == cap) == 0) store();
        else if (slot == cap) over.push(step << 10 | r);
        else store();
    }
    // Takes the least key out of the slots.  few: no lane of the wave has used more than four blocks (uniform).
    __device__ void take_slot(unsigned char *lds, bool few, bool supers) {
        const uint32_t slot = top & 1023u, block = slot / kPer;
        const uint32_t block_keys = keys + block * (kPer * 4), block_low = low + block * 4;
        at<uint32_t>(lds, keys + slot * 4) = kEmpty;
        at<uint32_t>(lds, block_low) = kEmpty;
        at<uint16_t>(lds, req + slot * 2) = (uint16_t)free_;
        asm volatile("" ::: "memory");
        auto min2 = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
        auto least = [&](const uint4 &v, uint32_t m) { return min2(min2(min2(min2(m, v.x), v.y), v.z), v.w); };
        uint4 k[kPer / 4];
#pragma unroll
        for (uint32_t i = 0; i < kPer / 4; ++i) k[i] = at<uint4>(lds, block_keys + i * 16);
        uint32_t others;                                // of the other blocks of the superblock
        if (few) {
            others = least(at<uint4>(lds, low), kEmpty);
        } else {
            const uint32_t group = low + block / kPer * 64;
            uint4 v[4];
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) v[i] = at<uint4>(lds, min2(group + i * 16, last_group));
            others = min2(least(v[1], least(v[0], kEmpty)), least(v[3], least(v[2], kEmpty)));
        }
        const uint32_t mine = min2(least(k[1], least(k[0], kEmpty)), least(k[3], least(k[2], kEmpty)));
        top = min2(mine, others);
        asm volatile("" ::: "memory");
        at<uint32_t>(lds, block_low) = mine;
        if (supers && super_) {
            at<uint32_t>(lds, super_ + block / kPer * 4) = top;
            asm volatile("" ::: "memory");
            top = least(at<uint4>(lds, super_), kEmpty);
            asm volatile("" ::: "memory");
        }
        free_ = slot;
    }
    // Takes the decoder out that leaves next and returns its request.  first: first_request() of this moment; spilled: some lane
    // of the wave has decoders beyond its slots (uniform).
    __device__ uint32_t take(unsigned char *lds, uint32_t first, bool few, bool supers, bool spilled) {
        if (!spilled) {
            take_slot(lds, few, supers);
            return first;
        }
        uint32_t r = first;
        if (top > over.top) {
            r = over.top & 1023u;
            over.pop();
        } else {
            take_slot(lds, few, supers);
        }
        return r;
    }
};

// The same as a heap, its first levels in LDS: for 64-bit keys, and for blocks whose lanes expect more decoders than LDS has
// slots for.
template <typename KeyT>
struct HeapQueue {
    LaneHeap<KeyT> heap;
    __device__ void init(unsigned char *lds, uint32_t groups, KeyT *mem) {
        heap.top = LaneHeap<KeyT>::kEmpty;
        heap.lds = (KeyT *)lds;
        heap.mem = mem;
        heap.cap = groups * kHeapWidth;
        heap.n = 0;
    }
    __device__ KeyT due() const { return heap.top >> 10; }
    __device__ void put(unsigned char *, KeyT step, uint32_t r, bool) { heap.push(step << 10 | r); }
    __device__ uint32_t take(unsigned char *, uint32_t, bool, bool, bool) {
        const uint32_t r = (uint32_t)(heap.top & 1023u);
        heap.pop();
        return r;
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

// Percentiles of simulated configurations that ended normally, a wave at a time.  TTFT of request i = first token time - arrival /
// rate; the values (absent requests, and those that arrive beyond the range of doubles, count as +inf) are sorted inside the wave's registers, R = 1, 2, 4, 8 or 16 per lane --
// as few as hold the trace -- by a bitonic network in which every compare-exchange puts the smaller value at the smaller
// index: element e = R * lane + register; a stage pairs e with e ^ m, which is another register of the same lane while m < R
// and the same-numbered (or mirrored) register of lane ^ (m / R) otherwise.  Then nearest-rank
// p50 = sorted[ceil(n/2) - 1] and p99 = sorted[ceil(0.99 n) - 1]; mean TPOT = mean over requests with more than
// one token of (finish - first token) / (tokens - 1).
// Bound by the vector ALU with 16 values (0.54 ms for 65 536 configurations with every exchange between lanes through
// LDS), by launch and reading with few (65 536 x 16 requests: a call 105 - 117 us, 540 - 580 us with 16 values for any trace).
constexpr uint32_t kMostPerLane = GUIDE_MAX_REQUESTS / kWave;   // 16

constexpr uint32_t top_bit(uint32_t x) { return x < 2 ? x : 2 * top_bit(x / 2); }
// compare-exchange inside a lane: the smaller value to the smaller register
__device__ inline void cx(double &a, double &b) {
    const double lo = fmin(a, b), hi = fmax(a, b);
    a = lo;
    b = hi;
}
// The value of lane ^ MASK, in the vector ALU where its patterns reach (0x1B reverses four lanes, 0x128 turns a row by eight).
template <uint32_t MASK>
__device__ inline double lane_xor(double x) {
    auto move = [](double y, auto ctrl) {
        const uint64_t b = (uint64_t)__double_as_longlong(y);
        const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
        constexpr int kCtrl = decltype(ctrl)::value;
        return __longlong_as_double((long long)((uint64_t)dpp_u32<kCtrl>(hi, hi) << 32 | dpp_u32<kCtrl>(lo, lo)));
    };
    if constexpr (MASK == 1) return move(x, std::integral_constant<int, 0xB1>{});
    else if constexpr (MASK == 2) return move(x, std::integral_constant<int, 0x4E>{});
    else if constexpr (MASK == 3) return move(x, std::integral_constant<int, 0x1B>{});
    else if constexpr (MASK == 4) return move(move(x, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{});
    else if constexpr (MASK == 7) return move(x, std::integral_constant<int, 0x141>{});
    else if constexpr (MASK == 8) return move(x, std::integral_constant<int, 0x128>{});
    else if constexpr (MASK == 15) return move(x, std::integral_constant<int, 0x140>{});
    else return __shfl_xor(x, (int)MASK, kWave);
}
// One stage of the network.  MASK: the xor mask on element numbers.
template <uint32_t MASK, uint32_t R>
__device__ inline void sort_stage(double (&v)[R], uint32_t lane) {
    if constexpr (MASK < R) {
#pragma unroll
        for (uint32_t r = 0; r < R; ++r)
            if ((r ^ MASK) > r) cx(v[r], v[r ^ MASK]);
    } else {
        constexpr uint32_t kLaneMask = MASK / R, kRegMask = MASK % R;       // kRegMask: 0 or R - 1 (mirror)
        // this lane holds the smaller indices of its pairs when the top bit of the lane mask is clear in its number
        constexpr uint32_t kTop = top_bit(kLaneMask);
        const bool keep_min = (lane & kTop) == 0;
        double o[R];
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) o[r] = lane_xor<kLaneMask>(v[r ^ kRegMask]);
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) v[r] = (o[r] < v[r]) == keep_min ? o[r] : v[r];      // (equal values: either)
    }
}
// Merge of sorted runs of K / 2 elements into sorted runs of K: the mirror stage, then halving distances.
template <uint32_t K, uint32_t R>
__device__ inline void sort_merge(double (&v)[R], uint32_t lane) {
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
template <uint32_t R>
__device__ inline double sorted_at(const double (&v)[R], uint32_t e) {
    double x = v[0];
#pragma unroll
    for (uint32_t r = 1; r < R; ++r) x = (e % R) == r ? v[r] : x;
    return __shfl(x, (int)(e / R), kWave);
}


// The times of configuration c's requests, element r * 64 + lane in register r (coalesced; the sort does not care where a value
// starts; past the last request: its times once more).
template <uint32_t R>
__device__ inline void load_times(const SimWs &ws, uint32_t n_req, uint32_t c, double (&f)[R], double (&n)[R]) {
    const uint32_t lane = threadIdx.x % kWave;
    const double *first = ws.first + (size_t)c * n_req, *fin = ws.fin + (size_t)c * n_req;
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = r * kWave + lane, j = i < n_req ? i : n_req - 1;
        f[r] = first[j];
        n[r] = fin[j];
    }
}
// TTFTs and the lane's sum of times per output token.  first(r, i), fin(r, i): times of request i, register r; request(i): request i
// of the trace.
template <uint32_t R, typename First, typename Fin, typename RequestOf>
__device__ inline double divide_times(uint32_t n_req, double rate, double (&v)[R], First &&first, Fin &&fin, RequestOf &&request) {
    double tp = 0.0;
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = r * kWave + threadIdx.x % kWave;
        double t = INFINITY;
        if (i < n_req) {
            const Request q = request(i);
            const double f = first(r, i);
            t = f - q.arrival / rate;
            t = t == t ? t : INFINITY;                      // (arrival / rate is infinite; the network cannot place a NaN)
            if (q.out > 1) tp += (fin(r, i) - f) / (double)(q.out - 1);
        }
        v[r] = t;
    }
    return tp;
}
// tp: the lane's sum, n_tp: the wave's requests with more than one token.
template <uint32_t R>
__device__ inline void sort_and_store(double (&v)[R], double tp, uint32_t n_tp, uint32_t n_req, uint32_t c, const guide_sim_out &out) {
    const uint32_t lane = threadIdx.x % kWave;
    for (int off = kWave / 2; off > 0; off >>= 1) tp += __shfl_xor(tp, off, kWave);
    sort_merge<2>(v, lane);
    sort_merge<4>(v, lane);
    sort_merge<8>(v, lane);
    sort_merge<16>(v, lane);
    sort_merge<32>(v, lane);
    sort_merge<64>(v, lane);
    if constexpr (R >= 2) sort_merge<128>(v, lane);
    if constexpr (R >= 4) sort_merge<256>(v, lane);
    if constexpr (R >= 8) sort_merge<512>(v, lane);
    if constexpr (R >= 16) sort_merge<1024>(v, lane);
    const double p50 = sorted_at(v, (n_req + 1) / 2 - 1);
    const double p99 = sorted_at(v, (uint32_t)((99ull * n_req + 99) / 100 - 1));
    if (lane == 0) {
        out.ttft_p50[c] = p50;
        out.ttft_p99[c] = p99;
        out.mean_tpot[c] = n_tp ? tp / (double)n_tp : 0.0;
    }
}

// A wave of the simulation kernel works out the percentiles of its configurations one after the other: the next one's times are
// requested while this one's are sorted.  next(c, rate): the next configuration (uniform), false when there is none.
template <uint32_t R, typename Next, typename RequestOf>
__device__ inline void wave_percentiles(const SimWs &ws, uint32_t n_req, const guide_sim_out &out, Next &&next, RequestOf &&request) {
    uint32_t c, c_next = 0;
    double rate, rate_next = 0.0;
    if (!next(c, rate)) return;
    double f[R], n[R];                                      // first token, last token
    load_times<R>(ws, n_req, c, f, n);
    for (;;) {                                              // (uniform)
        asm volatile("" ::: "memory");                      // (the trace is read again for every configuration: registers are for the times)
        const bool more = next(c_next, rate_next);
        double v[R];
        uint32_t n_tp = 0;
        const double tp = divide_times<R>(n_req, rate, v, [&](uint32_t r, uint32_t) { return f[r]; },
                                          [&](uint32_t r, uint32_t) {
                                              ++n_tp;
                                              return n[r];
                                          }, request);
        if (more) load_times<R>(ws, n_req, c_next, f, n);
        sort_and_store<R>(v, tp, wave_sum(n_tp), n_req, c, out);
        if (!more) return;
        c = c_next;
        rate = rate_next;
    }
}
// fn(integral_constant<values per lane>) for a trace of n_req requests
template <typename F>
__host__ __device__ inline void with_values_per_lane(uint32_t n_req, F &&fn) {
    if (n_req <= kWave) fn(std::integral_constant<uint32_t, 1>{});
    else if (n_req <= 2 * kWave) fn(std::integral_constant<uint32_t, 2>{});
    else if (n_req <= 4 * kWave) fn(std::integral_constant<uint32_t, 4>{});
    else if (n_req <= 8 * kWave) fn(std::integral_constant<uint32_t, 8>{});
    else fn(std::integral_constant<uint32_t, kMostPerLane>{});
}

// One wave per configuration, from position `from` of the launch order on (as given when it is not ordered).
template <uint32_t R>
__global__ __launch_bounds__(kPctBlock) void percentile_kernel(SimWs ws, const TraceDev *__restrict__ trace,
                                                               const double *__restrict__ rate_in, uint32_t n_req,
                                                               uint32_t n_cfg, guide_sim_out out, uint32_t from, bool ordered) {
    const uint32_t pos = from + blockIdx.x * (kPctBlock / kWave) + threadIdx.x / kWave;      // wave-uniform
    if (pos >= n_cfg) return;
    const uint32_t c = ordered ? (uint32_t)__builtin_amdgcn_readfirstlane((int)ws.perm[pos]) : pos;
    if (out.status[c] != GUIDE_SIM_OK) return;
    const double *first = ws.first + (size_t)c * n_req, *fin = ws.fin + (size_t)c * n_req;
    double v[R];
    uint32_t n_tp = 0;
    const double tp = divide_times<R>(n_req, rate_in[c], v, [&](uint32_t, uint32_t i) { return first[i]; },
                                      [&](uint32_t, uint32_t i) {
                                          ++n_tp;
                                          return fin[i];
                                      },
                                      [&](uint32_t i) { return Request{trace->arrival[i], 0u, trace->n_out[i]}; });
    sort_and_store<R>(v, tp, wave_sum(n_tp), n_req, c, out);
}

// What the host knows about the trace.
struct TraceSums {
    double out;             // generated tokens
    uint64_t tokens;        // prompt and generated tokens
    uint32_t longest;       // most prompt + generated tokens of one request
};

// One configuration per lane, `lanes` of them per wave (64 or 1).
// A round of the loop does at most one of each kind of thing (two of the second and third): one decoder leaves, one request
// enters, one prompt chunk is scheduled, a pass with prompts runs, one prompt turns into a decoder, a run of decode-only steps advances up to
// and including the step that retires the next decoder.  A lane with one event at a time takes one round per request;
// a lane with bursts takes a round per request as well, while the other lanes go on with theirs (loops over a burst
// make the whole wave wait for every lane's bursts in turn: 7000 loop turns per 1024 requests).
// A run's steps are advanced at once: a step's time is linear in the context while attention
// is bound by reading the cache at any context (nearly every lane), and the run's time a polynomial; otherwise the
// series of two pieces.  (One rounding of the clock per run, where a stepped clock has one per step: against 80-bit
// sums the first-token times of 150 requests of up to 1500 tokens, one after the other, are 3e-15 off, step by step 7.5e-14.)
// Which of the two ways a lane goes depends on its own configuration alone, never on its neighbours in the wave (which
// differ from call to call): the results of a configuration are the same bits in every list and every call.
// What bounds the kernel: a wave is a serial stream of instructions, four to six cycles each, and the waves of a compute unit
// share its fetch; the longest wave sets the time (65 536 configurations x 1024 requests: 2080 rounds of 4080 cycles, second
// admissions included; a wave has 673 000 vector, 163 000 scalar and 40 000 LDS instructions in the mean, 841 000, 184 000 and 47 000 with
// three quarters of the percentiles, and waits a third of its cycles).
// A call with percentiles: 3.74 ms, 3.60 ms under the other scheduler; 1999 x 97: 0.27 - 0.36 ms by the trace.  With all percentiles after the last
// wave's end 3.95, 3.97 and 0.31 - 0.42 ms: the waves of the first three parts of a list are done 0.5 - 1.3 ms before the dealt part's.
// (4-ary heaps in LDS, strides of 64 and 8 steps, forty branches a round: 7.7, 6.4 and 0.71 ms.)
// heap_bytes: LDS behind the staged trace, shared out among the block's lanes by what each expects.
// OWN: waves work out the percentiles of their own configurations, but for those of the dealt part.  (A variant of its own: with
// its registers allotted for both, the loop over the rounds takes 3 % longer.)
template <bool ADDITIVE, bool PREFILL_FIRST, typename KeyT, bool OWN>
__global__ __launch_bounds__(kSimBlock) void simulate_kernel(GridDesc g, const DevTables *__restrict__ tab,
                                                             const TraceDev *__restrict__ trace, uint32_t n_req,
                                                             const uint32_t *__restrict__ cfg_idx,
                                                             const double *__restrict__ rate_in, uint32_t n_cfg,
                                                             guide_sim_out out, SimWs ws, TraceSums sums, uint32_t lanes,
                                                             uint32_t heap_bytes, bool ordered) {
    // With 32-bit keys the whole trace is below 2^30 tokens, so blocks, budgets and steps fit 32 bits as well
    using Int = typename std::conditional<sizeof(KeyT) == 4, int32_t, long long>::type;
    constexpr Int kIntMax = sizeof(KeyT) == 4 ? (Int)0x7FFFFFFF : (Int)(1ll << 62);
    extern __shared__ __align__(16) unsigned char s_raw[];
    const Request *req = ((RequestsLds *)s_raw)->r;
    __shared__ uint4 s_total[kSimWaves];
    for (uint32_t i = threadIdx.x; i < n_req + 2; i += blockDim.x)
        ((RequestsLds *)s_raw)->r[i] = i < n_req ? Request{trace->arrival[i], trace->n_in[i], trace->n_out[i]}
                                                 : Request{__builtin_nan(""), 1, 1};
    for (uint32_t i = threadIdx.x; i < heap_bytes / 16; i += blockDim.x)
        ((uint4 *)(s_raw + sizeof(RequestsLds)))[i] = uint4{~0u, ~0u, ~0u, ~0u};
    const uint32_t wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, waves = blockDim.x / kWave;
    // Configurations that are ordered are so by their expected concurrency, and every wave of a block takes its lanes from
    // another part of them (of up to four): lanes of a wave behave alike, and every block has waves with short and with long queues.
    // The last part, where queues reach hundreds of keys, is dealt out lane by lane, so that no block has more of the longest
    // ones than its LDS holds; with one wave per block, that is all of them, whose lanes do not behave alike then.  In order / dealt,
    // 1024 requests: 5000 configurations 5.3 / 3.5 ms, 20 000 (two waves per block) 5.7 / 3.8 ms; 300 requests: 5000 1.11 / 1.12 ms,
    // 65 536 1.52 / 1.28 ms.  Every other part goes backwards: lists that are not ordered often repeat a pattern (of rates, say), and
    // the waves of a block would all meet its same place (2000 x 300 requests: 1 % more).
    const uint32_t in_part = wave & 1 ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
    const bool dealt = ordered && wave == waves - 1;
    const uint32_t pos = dealt ? (wave * lanes + lane) * gridDim.x + in_part : (wave * gridDim.x + in_part) * lanes + lane;
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

    // LDS segments of the queues, in units (blocks of slots; groups of siblings of a heap) of which every lane gets one.  A lane
    // can have at most min(sequence cap, requests) decoders (one of a heap's is in a register), and not many more than the pool
    // holds requests of average length.  Slots: a little more than the expected concurrency first (65 536
    // configurations, 1024 requests: the most decoders are within 1.44 times it, or 16 of it, in 99 of 100 lanes), what is
    // left over towards three times it; a heap: three times it, or less by the same factor in all lanes, what is left over
    // towards the most.
    // Returns false when the slots' wants do not fit: then a heap is the better queue, which finds the decoders beyond its
    // segment in fewer accesses (lanes of 700 - 1024 decoders, in ms, heap / slots: 65 536 7.8 - 8.3 / 16.6 - 17.0, 16 000 3.9 - 4.4 /
    // 5.7 - 6.2, 3000 3.8 - 4.5 / 5.0 - 5.7).  To be called by the whole block.
    uint32_t n_units = 0, off = 0;
    auto allot = [&](auto tag) {
        constexpr bool kSlots = decltype(tag)::value;
        constexpr uint32_t kUnit = kSlots ? SlotQueue::kPer : kHeapWidth;
        constexpr uint32_t kFirst = kSlots ? SlotQueue::kFirstBytes : kHeapWidth * sizeof(KeyT);
        constexpr uint32_t kMore = kSlots ? SlotQueue::kMoreBytes : kHeapWidth * sizeof(KeyT);
        auto bytes_of = [](uint32_t n) { return kSlots ? SlotQueue::bytes(n) : n * kFirst; };
        auto units = [](uint32_t x) { return x ? (x + kUnit - 1) / kUnit : 1u; };
        const uint32_t most = (max_seqs < n_req ? max_seqs : n_req) - (kSlots ? 0u : 1u);
        const float mean_blocks = (float)sums.tokens / (float)n_req / (float)dblk.d + 0.5f;
        const float pool = fminf(1.5f * (float)n_blk / mean_blocks + 4.0f, 2048.0f);
        uint32_t full = units(most < (uint32_t)pool ? most : (uint32_t)pool), want = full;
        if (ordered) {
            const float expected = expected_of(alive ? ws.bucket[c] : 0u);
            const uint32_t likely = units((uint32_t)(1.25f * expected) + 14u), enough = units((uint32_t)(3.0f * expected) + 16u);
            if (kSlots) full = enough < full ? enough : full;
            want = kSlots ? (likely < full ? likely : full) : (enough < full ? enough : full);
        }
        // the bytes of the wants, the units beyond them, and theirs beyond the first
        const uint32_t wave_bytes = wave_sum(alive ? bytes_of(want) : 0u), wave_extra = wave_sum(alive ? full - want : 0u);
        const uint32_t wave_more = wave_sum(alive ? want - 1u : 0u);
        if (lane == 0) s_total[wave] = uint4{wave_bytes, wave_extra, wave_more, 0u};
        __syncthreads();                                // the trace and the empty segments are staged as well
        uint32_t total = 0, extra = 0, more = 0;
        for (uint32_t w = 0; w < waves; ++w) {
            total += s_total[w].x;
            extra += s_total[w].y;
            more += s_total[w].z;
        }
        __syncthreads();
        if (kSlots && total > heap_bytes) return false;
        n_units = want;
        if (total > heap_bytes)                         // (heap_bytes holds a unit for every lane in use)
            n_units = 1u + (uint32_t)((double)(want - 1u) * ((double)(heap_bytes - waves * lanes * kFirst) / (double)kMore / (double)more));
        else if (extra)                                 // (a lane's segment grows by kMore a unit, and by 48 bytes at most beside)
            n_units = want + (uint32_t)((double)(full - want) *
                                        fmin((double)(heap_bytes - total) / (double)(kMore + 48u) / (double)extra, 1.0));
        n_units = alive ? n_units : 0u;
        const uint32_t mine = alive ? bytes_of(n_units) : 0u;
        const uint32_t incl = wave_scan_sum(mine);
        if (lane == kWave - 1) s_total[wave].x = incl;
        __syncthreads();
        off = sizeof(RequestsLds) + incl - mine;
        for (uint32_t w = 0; w < wave; ++w) off += s_total[w].x;
        return true;
    };
    // attention bound by reading the cache at every context: step times are linear (in every lane: wave_linear, which only
    // leaves work out that changes nothing in such a lane)
    const bool lane_linear = ADDITIVE || lt.c_att <= lt.m_att_k;
    const bool wave_linear = ADDITIVE || __ballot(alive && !lane_linear) == 0;
    bool ended = false;                                             // the lane's simulation has ended normally
    auto simulate = [&](auto &queue) {
        constexpr bool kSlots = std::is_same<decltype(queue), SlotQueue &>::value;
        if (!alive) return;

        bool few = true, supers = false;                        // (SlotQueue: uniform)
        if constexpr (kSlots) supers = __ballot(queue.super_ != 0) != 0;
        double *first = ws.first + (size_t)c * n_req, *fin = ws.fin + (size_t)c * n_req;

        // arrival / rate: the reciprocal's product with one correction step rounds as the division does, unless the quotient lies
        // within 2^-50 units of its last place of a rounding boundary; rates and traces at the ends of the range are divided
        const double last_arrival = req[n_req - 1].arrival;
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

        double now = 0.0, s_ctx = 0.0;                          // s_ctx: total context, an integer far below 2^53
        // prompts [comp, next) are admitted and have not emitted their first token; the next one to schedule is h, of which
        // `done` tokens have been computed; pend: prompts from comp on whose last chunk was in the pass just run
        uint32_t next = 0, comp = 0, h = 0, done = 0, pend = 0, n_dec = 0, n_done = 0;
        double c_T = 0.0, c_Q = 0.0, c_K = 0.0;                 // chunks scheduled for the next pass: tokens, workload, context
        uint32_t chunks = 0, n_full = 0;                        // their number, and prompts that they complete
        Int used = 0;                                           // their tokens
        uint64_t n_rs = 0;
        typename std::conditional<sizeof(KeyT) == 4, uint32_t, uint64_t>::type step = 0;       // (every step consumes a token of some request)
        KeyT dstep = 0;                                         // steps in which decoders ran
        Int free_blk = n_blk;
        uint32_t status = GUIDE_SIM_OK;
        const uint64_t step_bound = (uint64_t)n_req + sums.tokens;      // every step consumes at least one token of some request
        double arr_next = arrival_of(req[0].arrival);           // arrival time of request `next`, no number when none is left
        Int need_next = blocks_of(req[0].in + req[0].out);

        // A round costs its instructions, four to six cycles each, and forty for every branch that lanes take differently: what
        // is cheap is computed in all lanes and selected.
        for (;;) {
            // everything that the steps below read from LDS, requested together
            const Request q_new = req[next + 1], q_h = req[h], q_comp = req[comp];
            const uint32_t in_next = PREFILL_FIRST ? req[h + 1].in : 0u;
            uint32_t first_r = 0;
            bool spilled = false;
            if constexpr (kSlots) {
                first_r = queue.first_request(s_raw);
                spilled = __ballot(queue.over.n != 0) != 0;
                few = few && __ballot(queue.used > 4u * SlotQueue::kPer) == 0;
            }
            // 1. a decoder that has emitted its last token leaves (with none, the next one to leave is beyond every step)
            const bool leave = queue.due() == dstep;
            if (leave) {
                const uint32_t r = queue.take(s_raw, first_r, few, supers, spilled);
                const uint32_t tokens = req[r].in + req[r].out;
                free_blk += blocks_of(tokens);
                --n_dec;
                s_ctx -= (double)tokens;
                ++n_done;
                fin[r] = now;
            }
            if (n_done == n_req) break;
            // 2. idle: jump to the next arrival
            uint32_t active = (next - comp) + n_dec;
            now = active == 0 && arr_next > now ? arr_next : now;
            // 3. and 4. once for all lanes, and once more while some lane of the wave is in a burst of arrivals (65 536
            // configurations: 4.12 instead of 4.65 ms; up to three more times 4.9: the other lanes wait)
            bool enter = false, room = false, sched = false, whole = false;
            const bool leaving = queue.due() == dstep;
            Request q_n = q_new, q_c = q_h;
            uint32_t in_after = in_next;
            auto admit_and_schedule = [&]() {
                // 3. FCFS admission of one request, if it can enter.  (Decoders that still have to leave, or prompts that turn into
                // decoders, only make room: whoever enters before would enter after.)
                enter = active < max_seqs && arr_next <= now && need_next <= free_blk;
                const double arr_new = arrival_of(q_n.arrival);
                const Int need_new = blocks_of(q_n.in + q_n.out);
                free_blk -= enter ? need_next : 0;
                next += enter ? 1u : 0u;
                active += enter ? 1u : 0u;
                arr_next = enter ? arr_new : arr_next;
                need_next = enter ? need_new : need_next;
                room = active < max_seqs && need_next <= free_blk;      // for the next one, when it has arrived
                // 4. schedule one prompt chunk.  Split-fuse: the budget that the decoders leave, whose number is final once nobody
                // leaves or joins any more; a whole prompt may go in before when it fits for sure.  Prefill-first:
                // whole prompts, as many as fit the budget, the first always.
                const Int rem = (Int)(q_c.in - done);
                const Int left = PREFILL_FIRST ? budget_full - used : budget_full - (Int)(n_dec + pend) - used;
                const bool fits = PREFILL_FIRST ? (chunks == 0 || rem <= left) : (rem <= left || (left > 0 && !leaving && pend == 0));
                sched = h < next && fits;
                const Int ch = !sched ? 0 : PREFILL_FIRST || rem < left ? rem : left;
                whole = sched && ch == rem;
                {
                    const uint32_t to = done + (uint32_t)ch;
                    const double C = (double)ch, ctx = (double)to;
                    used += ch;
                    c_T += C;
                    c_Q = fma(C, ctx, c_Q);
                    c_K += sched ? ctx : 0.0;
                    chunks += sched ? 1u : 0u;
                    n_full += whole ? 1u : 0u;
                    h += whole ? 1u : 0u;
                    done = whole ? 0u : to;
                }
            };
            admit_and_schedule();
            bool moved = enter || sched;
            if (__ballot((enter && room && arr_next <= now) || (whole && h < next)) != 0) {
                q_n = req[next + 1];
                q_c = req[h];
                if (PREFILL_FIRST) in_after = req[h + 1].in;
                admit_and_schedule();
                moved = moved || enter || sched;
            }
            // 5. a pass with prompts, once nothing is left to be done before it: one token per decoder (prefill-first:
            // the decoders pause) and the scheduled chunks
            const bool more = h < next && (PREFILL_FIRST ? (Int)(whole ? in_after : q_c.in) <= budget_full - used
                                                         : budget_full - (Int)n_dec - used > 0);
            const bool pass = comp < next && !leaving && pend == 0 && !more && !(room && arr_next <= now);
            if (pass) {
                const double d = PREFILL_FIRST ? 0.0 : (double)n_dec, ctx = PREFILL_FIRST ? 0.0 : s_ctx;
                const double T = c_T + d, Q = c_Q + ctx, K = c_K + ctx;
                now += pass_base<ADDITIVE>(lt, T, d + (double)n_full) +
                       op_time<ADDITIVE>(Q * lt.c_att, fma(K, lt.m_att_k, T * lt.m_att_t));
                ++step;
                n_rs += chunks;
                if (!PREFILL_FIRST) {
                    n_rs += n_dec;
                    dstep += n_dec > 0 ? 1 : 0;
                    s_ctx += d;
                }
                pend = n_full;
                c_T = c_Q = c_K = 0.0;
                chunks = n_full = 0;
                used = 0;
            }
            // 6. a prompt completed in the last pass emits its first token.  (With a single token to generate it leaves in the next
            // round, at the same moment.)
            const bool join = pend > 0;
            if (join) {
                first[comp] = now;
                queue.put(s_raw, dstep + (KeyT)(q_comp.out - 1), comp, supers);
                ++n_dec;
                s_ctx += (double)(q_comp.in + 1);
                ++comp;
                --pend;
            }
            // 7. run of decode-only steps: no prompt is waiting, and nothing changes until the first decoder emits its
            // last token or a request that could be admitted arrives.
            const KeyT end_step = queue.due();
            const bool can_admit = next < n_req && n_dec < max_seqs && need_next <= free_blk;
            const bool go = comp == next && n_dec > 0 && end_step != dstep && !(can_admit && arr_next <= now);
            if (go) {
                const double T = (double)n_dec;
                const uint32_t total = (uint32_t)(end_step - dstep);     // steps up to the one that retires a decoder
                // time of a step at context c: base + max(c_att c, m_att_k c + T m_att_t)
                const double base = pass_base<ADDITIVE>(lt, T, T), base_m = fma(T, lt.m_att_t, base);
                const double slope = ADDITIVE ? lt.c_att + lt.m_att_k : lt.m_att_k;
                const double h_T = 0.5 * T, ctx0 = s_ctx - h_T;
                // The least r with arr_next <= now + time(r), total when there is none below it.  time(r) = p r + q r^2 up to
                // rounding on the side that the run starts on; its root in single precision is the first guess.
                const bool arith = !wave_linear && !lane_linear && fma(s_ctx, lt.c_att, base) >= fma(s_ctx, slope, base_m);
                const double sl = arith ? lt.c_att : slope;
                const float rem_t = (float)(arr_next - now), q = (float)(sl * h_T), p = (float)fma(sl, ctx0, arith ? base : base_m);
                const float root = ceilf(2.0f * rem_t * __builtin_amdgcn_rcpf(p + __builtin_amdgcn_sqrtf(fmaf(p, p, 4.0f * q * rem_t))));
                const float guess = can_admit && root < (float)total ? (root >= 1.0f ? root : 1.0f) : (float)total;
                uint32_t run = 0;
                if (wave_linear || lane_linear) {
                    auto time_of = [&](double r) { return r * fma(slope, fma(h_T, r, ctx0), base_m); };
                    // the guess is right or one off nearly always, so its neighbours are looked at side by side
                    // (no number where no arrival ends the run: at or before nothing, an infinite clock included)
                    const double G = (double)guess, stop = can_admit ? arr_next : __builtin_nan("");
                    const bool far_below = stop <= now + time_of(G - 2.0), below = stop <= now + time_of(G - 1.0);
                    const bool here = stop <= now + time_of(G), above = stop <= now + time_of(G + 1.0);
                    run = (uint32_t)guess + (below ? ~0u : 0u) + (here ? 0u : 1u);
                    run = run < total ? run : total;
                    if (far_below || !(here || above || run == total)) run = least_steps(now, arr_next, total, guess, time_of);
                    now += time_of((double)run);
                } else {
                    auto time_of = [&](double r) {
                        return fma(r, base, attention_series<ADDITIVE>(lt.c_att, lt.m_att_k, T * lt.m_att_t, s_ctx - T, T,
                                                                       fast_recip(T), r));
                    };
                    run = can_admit ? least_steps(now, arr_next, total, guess, time_of) : total;
                    now += time_of((double)run);
                }
                step += run;
                dstep += (KeyT)run;
                n_rs += (uint64_t)run * n_dec;
                s_ctx = fma((double)run, T, s_ctx);
            }
            if (step > step_bound || !(leave || moved || pass || join || go)) {        // a round always moves something
                status = GUIDE_SIM_INTERNAL;
                break;
            }
        }

        out.tokens_s[c] = status == GUIDE_SIM_OK ? sums.out / (now - req[0].arrival / rate) : 0.0;
        if (OWN) ended = status == GUIDE_SIM_OK;
        out.status[c] = status;
        out.n_steps[c] = step;
        out.n_request_steps[c] = n_rs;
        if (status != GUIDE_SIM_OK) {
            out.ttft_p50[c] = INFINITY; out.ttft_p99[c] = INFINITY; out.mean_tpot[c] = INFINITY;
        }
    };

    KeyT *mem = (KeyT *)(ws.heap + (size_t)pos * n_req);
    bool slots = false;                                             // (block-uniform)
    if constexpr (sizeof(KeyT) == 4) {
        slots = allot(std::true_type{});
        if (slots) {
            SlotQueue queue;
            queue.init(off, n_units, mem);
            simulate(queue);
            if constexpr (!OWN) return;
        }
    }
    if (!slots) {
        allot(std::false_type{});
        HeapQueue<KeyT> queue;
        queue.init(s_raw + off, n_units, mem);
        simulate(queue);
    }
    if constexpr (!OWN) return;

    // Percentiles, by the waves that are done before the longest ones: those of the dealt part are left to a kernel
    // that has the whole chip for them.
    if (dealt) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");          // the lanes read each other's times
    uint64_t left = __ballot(ended);
    auto next_ended = [&](uint32_t &cfg, double &r) {
        if (left == 0) return false;
        const int j = __ffsll((long long)left) - 1;
        left &= left - 1;
        cfg = (uint32_t)__builtin_amdgcn_readlane((int)c, j);
        const uint64_t bits = (uint64_t)__double_as_longlong(rate);
        r = __longlong_as_double((long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(bits >> 32), j) << 32 |
                                             (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, j)));
        return true;
    };
    with_values_per_lane(n_req, [&](auto per_lane) {
        wave_percentiles<decltype(per_lane)::value>(ws, n_req, out, next_ended, [&](uint32_t i) { return req[i]; });
    });
}

}  // namespace

size_t simulate_workspace_bytes(uint32_t n_cfg, uint32_t n_req) {
    return (size_t)n_cfg * n_req * 24 + (size_t)n_cfg * 8 + kKeyBins * 4 + 256;
}

hipError_t launch_simulate(const GridDesc &g, const DevTables *tab, const TraceDev *trace, uint32_t n_req,
                           const uint32_t *cfg_idx, const double *rate, uint32_t n_cfg, bool additive,
                           bool prefill_first, const guide_sim_out &out, void *ws_, hipStream_t stream,
                           double sum_in, double sum_out, uint32_t longest,
                           double unit_rate) {
    const SimWs ws = sim_ws(ws_, n_cfg, n_req);
    const TraceSums sums{sum_out, (uint64_t)(sum_in + sum_out), longest};
    // Lanes in use per wave and waves per block.  The waves of a compute unit share its instruction fetch, so few waves are
    // fast ones: short lists take a lane per wave and a wave per block, and beyond that (a block per compute unit) eight
    // waves; long ones 64 lanes (a few lanes leave out few of a round's sections) and as few waves per block as still give every
    // compute unit one block, also for the LDS that its lanes share.  In us, 97 / 300 requests, waves x lanes: 300 configurations
    // 1 x 1 302 / 777, 8 x 1 462 / 1179, 1 x 64 443 / 1095; 600: 368 / 969, 382 / 1014, 451 / 1119; 1000: 8 x 1 364 / 925, 1 x 64 461 / 1143;
    // 2000: 352 / 886, 468 / 1182; 4000: 8 x 1 572 / 1482, 1 x 16 509 / 1247, 1 x 64 487 / 1192; 16 000: 1 x 64 572 / 1288, 2 x 32 584 / 1321.
    // In ms, 1024 requests: 500 1 x 1 3.0, 8 x 1 4.3, 1 x 64 3.4; 1000 8 x 1 3.7, 1 x 64 3.4; 2000 3.4, 3.5; 2500 5.9, 3.5.
    const uint32_t cus = device_cus(), lanes = n_cfg <= 8 * cus ? 1 : kWave, full_waves = (n_cfg - 1) / (kWave * cus) + 1;
    const uint32_t waves = lanes == 1 ? (2 * n_cfg <= 5 * cus ? 1 : 8) : (full_waves < 4 ? full_waves : 4);
    const uint32_t per_block = waves * lanes;
    // LDS beyond the staged trace holds heap nodes of the block's lanes; 32-bit keys when every finishing step
    // (at most the trace's generated tokens) fits 22 bits and the trace's tokens fit 30
    const bool key32 = sum_out < 4194303.0 && sum_in < 1073700000.0;
    int dev = 0, lds_max = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return e;
    const size_t staged = sizeof(RequestsLds), fixed = staged + kSimStaticLds;
    const size_t unit = key32 ? SlotQueue::kFirstBytes : kHeapWidth * sizeof(uint64_t);
    if ((size_t)lds_max < fixed + per_block * unit) return hipErrorInvalidValue;
    size_t heap_bytes = (size_t)lds_max - fixed;
    // no lane needs more
    const size_t most = per_block * (key32 ? SlotQueue::bytes((n_req + SlotQueue::kPer - 1) / SlotQueue::kPer)
                                           : (n_req + 2 * kHeapWidth) * sizeof(uint64_t));
    const bool all_fit = most <= heap_bytes;
    heap_bytes = all_fit ? most : heap_bytes;
    heap_bytes -= heap_bytes % 16;
    const size_t lds_bytes = staged + heap_bytes;
    const dim3 grid((n_cfg + per_block - 1) / per_block), block(waves * kWave);
    const dim3 ogrid((n_cfg + kOrderBlock - 1) / kOrderBlock), oblock(kOrderBlock);
    const bool ordered = lanes > 1 && (waves > 1 ? n_req >= kOrderRequests : !all_fit);
    if (ordered) {
        hipLaunchKernelGGL(sim_order_clear_kernel, dim3(1), dim3(kKeyBins), 0, stream, ws);
        if (additive)
            hipLaunchKernelGGL(sim_order_count_kernel<true>, ogrid, oblock, 0, stream, g, tab, n_req, cfg_idx, rate, n_cfg, ws, sum_in, sum_out,
                               unit_rate);
        else
            hipLaunchKernelGGL(sim_order_count_kernel<false>, ogrid, oblock, 0, stream, g, tab, n_req, cfg_idx, rate, n_cfg, ws, sum_in, sum_out,
                               unit_rate);
        hipLaunchKernelGGL(sim_order_scan_kernel, dim3(1), dim3(kKeyBins), 0, stream, ws);
        hipLaunchKernelGGL(sim_order_scatter_kernel, ogrid, oblock, 0, stream, n_cfg, ws);
    }
    // Who works out the percentiles.  In blocks of four waves, those that are done before the longest ones: where the trace is long enough, and
    // fills the values that are sorted well enough (256 from 129 requests on, 512 from 257 on, ..), that working them out one after the other is done
    // by then.  In us, by the waves / by a kernel: 65 536 x 64 304 / 281, x 96 427 / 423, x 128 557 / 580, x 129 612 / 592, x 150 and 160
    // 1 % less, x 192 5 % less, x 300 1257 / 1306, x 600 2410 / 2490, x 1024 3743 / 3930; 80 000 x 129 and 140 5 % more, x 160 1.5 % more, x 180
    // 1 % less; 300 000 x 129 1 % more, x 150 3 % less.  With fewer blocks than compute units: 49 153 x 257 and 513 1.3 % more, x 288 and 576 1 %
    // less.  Two or three waves: 20 000 x 600 2375 / 2288, 49 000 x 1024 3828 / 3865.  Waves of a lane each do it themselves, which saves the launch: 2000 x 16
    // 56 / 67, 1999 x 97 285 / 327, 1500 x 1024 2967 / 3240, 300 and 512 configurations within 3 % either way from 200 requests on; but a wave that has a compute unit to itself has nobody to
    // wait for, and the loop over the rounds is 2 - 3 % slower in this variant: 256 x 16 50 / 54, x 60 153 / 154, x 300 724 / 708, x 1024 2440 / 2334.
    uint32_t sorted = kWave;                            // values that are sorted
    while (sorted < n_req) sorted *= 2;
    const uint32_t sixteenths = sorted == 4 * kWave ? 10u : sorted > 4 * kWave && grid.x < cus ? 9u : 0u;   // of them at least are requests
    const bool own_percentiles = lanes == 1 ? n_cfg > cus || n_req <= kWave
                                            : ordered && waves > 3 && n_req >= 128 && 16 * n_req >= sixteenths * sorted;
    const int variant = (additive ? 4 : 0) | (prefill_first ? 2 : 0) | (key32 ? 1 : 0);
#define GUIDE_SIM(A, P, K32)                                                                                       \
    case ((A ? 4 : 0) | (P ? 2 : 0) | (K32 ? 1 : 0)): {                                                             \
        using Key = std::conditional<K32, uint32_t, uint64_t>::type;                                                \
        auto kern = own_percentiles ? simulate_kernel<A, P, Key, true> : simulate_kernel<A, P, Key, false>;         \
        e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);    \
        if (e != hipSuccess) return e;                                                                              \
        hipLaunchKernelGGL(kern, grid, block, lds_bytes, stream, g, tab, trace, n_req, cfg_idx, rate, n_cfg, out, ws, \
                           sums, lanes, (uint32_t)heap_bytes, ordered);                                             \
        break;                                                                                                      \
    }
    switch (variant) {
        GUIDE_SIM(false, false, false) GUIDE_SIM(false, false, true) GUIDE_SIM(false, true, false) GUIDE_SIM(false, true, true)
        GUIDE_SIM(true, false, false) GUIDE_SIM(true, false, true) GUIDE_SIM(true, true, false) GUIDE_SIM(true, true, true)
    }
#undef GUIDE_SIM
    // Percentiles that the simulation kernel has left
    const uint32_t from = !own_percentiles ? 0u : ordered ? (waves - 1) * lanes * grid.x : n_cfg;
    if (from < n_cfg) {
        const dim3 pgrid((n_cfg - from + kPctBlock / kWave - 1) / (kPctBlock / kWave));
        with_values_per_lane(n_req, [&](auto per_lane) {
            hipLaunchKernelGGL((percentile_kernel<decltype(per_lane)::value>), pgrid, dim3(kPctBlock), 0, stream, ws,
                               trace, rate, n_req, n_cfg, out, from, ordered);
        });
    }
    return hipGetLastError();
}

}  // namespace guide
