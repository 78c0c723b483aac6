// Selection kernels: constrained per-group top-k by (objective, row) order and
// the two-objective Pareto front.  Reductions run in registers and across lanes
// in the vector ALU, then through LDS per block, then in a small second pass over
// the block partials.
//
// Paper: the simulator evaluates every configuration and keeps the one(s) with
// the least total time (Simulating Hybrid Parallelism); the engine keeps the top
// three by inference time / throughput (Inference Engine, Step 2).
#include "kernels.hpp"
#include "reduce.hpp"
#include "select_shared.hpp"

#include <hip/hip_ext.h>

#include <cstring>
#include <type_traits>

namespace guide {

namespace {

constexpr int kWaves = kBlock / kWave;

struct RowFilter {
    const uint8_t *feasible;
    uint32_t n_con;
    const double *col[GUIDE_MAX_CONSTRAINTS];
    double cap[GUIDE_MAX_CONSTRAINTS];
};

// All loads of a row are issued unconditionally (index clamped when the row is
// past the end) and nothing is computed from them here, so that many rows can be
// in flight while the kernel does other work; row_of() turns the loaded values
// into the row's coordinates and its filter verdict.
// MAXC: constraint columns the kernel variant can hold (n_con <= MAXC); variants with fewer keep
// fewer registers busy per row in flight.
template <uint32_t MAXC>
struct RawRow {
    double x, y;
    double c[MAXC ? MAXC : 1];
    uint8_t fe;
    bool valid;
};
struct Row {
    double x, y;
    bool pass;
};
template <bool WITH_Y, uint32_t MAXC>
__device__ inline RawRow<MAXC> load_raw(const double *__restrict__ x, const double *__restrict__ y, const RowFilter &f,
                                        uint32_t i, uint32_t n) {
    RawRow<MAXC> r;
    r.valid = i < n;
    const uint32_t j = r.valid ? i : 0;
    r.x = x[j];
    r.y = WITH_Y ? y[j] : 0.0;
    r.fe = f.feasible ? f.feasible[j] : (uint8_t)1;
#pragma unroll
    for (uint32_t k = 0; k < MAXC; ++k) r.c[k] = k < f.n_con ? f.col[k][j] : 0.0;
    return r;
}
template <bool WITH_Y, uint32_t MAXC>
__device__ inline Row row_of(const RawRow<MAXC> &w, const RowFilter &f) {
    bool ok = w.valid && w.fe != 0 && (w.x == w.x) && (!WITH_Y || w.y == w.y);
#pragma unroll
    for (uint32_t k = 0; k < MAXC; ++k)
        if (k < f.n_con) ok = ok && (w.c[k] <= f.cap[k]);
    return Row{w.x, w.y, ok};
}
template <bool WITH_Y, uint32_t MAXC>
__device__ inline Row load_row(const double *__restrict__ x, const double *__restrict__ y, const RowFilter &f,
                               uint32_t i, uint32_t n) {
    return row_of<WITH_Y, MAXC>(load_raw<WITH_Y, MAXC>(x, y, f, i, n), f);
}
// Launches fn.template operator()<MAXC>() for the least supported MAXC >= n_con.
template <typename F>
void with_max_constraints(uint32_t n_con, F &&fn) {
    if (n_con == 0) fn(std::integral_constant<uint32_t, 0>{});
    else if (n_con == 1) fn(std::integral_constant<uint32_t, 1>{});
    else fn(std::integral_constant<uint32_t, GUIDE_MAX_CONSTRAINTS>{});
}

// Rows are dealt to blocks in chunks of `chunk` rows (a multiple of kBlock): chunk c goes to block c % gridDim.x.
// The hardware deals blocks to the dies' L2 caches round robin, so with a grid that is a multiple of the number of
// dies, chunk c is read through the same L2 as by any other kernel that deals the same chunks the same way -- in
// particular the evaluation kernel that writes them, which then finds no copies of its lines in other L2s.
// A block walks its chunks in batches of kBlock * U rows (the last batch of a chunk may be partial), U = rows per
// thread in flight: 8, or 6 when that divides the chunk evenly and 8 does not.
constexpr uint32_t kUnroll = 8;
constexpr uint32_t kDefaultChunk = kBlock * kUnroll;
template <uint32_t U>
struct ChunkWalk {
    uint32_t chunk, n, n_blocks, c;
    uint64_t base, end;             // current batch starts at `base`; its chunk ends at `end` (exclusive)
    __device__ ChunkWalk(uint32_t chunk_, uint32_t n_, uint32_t n_blocks_)
        : chunk(chunk_), n(n_), n_blocks(n_blocks_), c(blockIdx.x) { enter(); }
    __device__ void enter() {
        base = (uint64_t)c * chunk;
        end = base + chunk < n ? base + chunk : n;
    }
    __device__ bool live() const { return base < n; }
    __device__ void next() {
        base += kBlock * U;
        if (base >= end) {
            c += n_blocks;
            enter();
        }
    }
};

RowFilter make_filter(const guide_select_spec &s) {
    RowFilter f;
    f.feasible = s.feasible;
    f.n_con = s.n_constraints;
    for (uint32_t c = 0; c < GUIDE_MAX_CONSTRAINTS; ++c) {
        f.col[c] = c < s.n_constraints ? s.constraints[c].column : nullptr;
        f.cap[c] = c < s.n_constraints ? s.constraints[c].cap : 0.0;
    }
    return f;
}

// Blocks of a streaming pass over n rows.  Top-k passes: up to four per compute unit.  The Pareto filter pass:
// three per compute unit -- every block loads a 32 KB table of sample rows and ends with a block-level top-k
// merge, which with more blocks costs more than the extra blocks hide (1.9M rows in chunks of 1536: 13.8 us with
// 768 blocks, 14.5 with 1024, 15.0 with 624, 15.1 - 15.6 with 512, 16.2 with 416).
uint32_t blocks_for(uint64_t n) {
    uint64_t need = (n + kBlock - 1) / kBlock;
    if (need == 0) need = 1;
    return (uint32_t)(need < kSelBlocks ? need : kSelBlocks);
}
uint32_t pareto_blocks(uint64_t n) {
    uint64_t need = (n + kBlock - 1) / kBlock, cap = 3 * (uint64_t)device_cus();
    if (need == 0) need = 1;
    cap = cap < kSelBlocks ? cap : kSelBlocks;
    return (uint32_t)(need < cap ? need : cap);
}

// ------------------------------------------------------- top-k, one group

// Independent work of another selection that rides along with a launch as extra blocks, so that it
// does not pay for a launch of its own.  SampleRider: the row sample of a Pareto selection
// (kSampleBlocks blocks after the host kernel's own).  MergeRider: the merge of top-k block partials
// (one block).  n_blocks = 0 / on = 0: none.
struct SampleRider {
    uint32_t on;
    const double *x, *y;
    RowFilter f;
    SelectScratch *sc;
};
struct MergeRider {
    Top1Ws w;
    uint32_t n_blocks, k, K;       // K: pairs per block partial (1 .. 4)
    uint64_t *out_idx;
    double *out_val;
    uint64_t *out_cnt;
};
__device__ void pareto_prepare_body(uint32_t block, const double *__restrict__ x, const double *__restrict__ y,
                                    const RowFilter &f, uint32_t n, SelectScratch *sc);

// One pass over the rows: every lane keeps its K best, the block merges them.  Blocks
// [0, n_row_blocks) take the rows.
template <int K, uint32_t MAXC, uint32_t U>
__global__ __launch_bounds__(kBlock) void topk_pass_kernel(const double *__restrict__ obj, RowFilter f, uint32_t n,
                                                           Top1Ws w, uint32_t n_row_blocks, SampleRider sample,
                                                           uint32_t chunk) {
    if (blockIdx.x >= n_row_blocks) {
        pareto_prepare_body(blockIdx.x - n_row_blocks, sample.x, sample.y, sample.f, n, sample.sc);
        return;
    }
    __shared__ Pair s_pairs[kWaves][K];
    __shared__ uint64_t s_cnt[kWaves];
    TopList<K> l;
    l.init();
    uint32_t cnt = 0;                                   // rows of one lane: fewer than 2^32
    for (ChunkWalk<U> cw(chunk, n, n_row_blocks); cw.live(); cw.next()) {
        const uint32_t base = (uint32_t)cw.base + threadIdx.x, lim = (uint32_t)cw.end;
        Row r[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) r[u] = load_row<false, MAXC>(obj, nullptr, f, base + u * kBlock, lim);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (r[u].pass) {
                ++cnt;
                l.insert_ascending(Pair{key_of(r[u].x), base + u * kBlock});
            }
        }
    }
    const uint32_t wave_cnt = wave_sum(cnt);             // a wave's rows: fewer than 2^32 as well
    if (threadIdx.x % kWave == 0) s_cnt[threadIdx.x / kWave] = wave_cnt;
    block_topk<K, kWaves>(l, s_pairs, [&](int r, const Pair &p) {
        w.key[(size_t)blockIdx.x * K + r] = p.key;
        w.idx[(size_t)blockIdx.x * K + r] = p.idx;
    });                                                 // (contains the barrier that publishes s_cnt)
    if (threadIdx.x == 0) {
        uint64_t c = 0;
        for (int wv = 0; wv < kWaves; ++wv) c += s_cnt[wv];
        w.cnt[blockIdx.x] = c;
    }
}

// One block of NT threads: the K least of the block partials, and the total count.
constexpr uint32_t kMergeThreads = 512;
template <int K, uint32_t NT>
__device__ inline void topk_merge_body(Top1Ws w, uint32_t n_blocks, uint32_t k, uint64_t *out_idx, double *out_val,
                                       uint64_t *out_cnt) {
    constexpr int kNW = NT / kWave;
    __shared__ Pair s_pairs[kNW][K];
    __shared__ uint64_t s_cnt[kNW];
    constexpr uint32_t kPer = kSelBlocks * K / NT;       // all loads first: one memory latency
    Pair c[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        const uint32_t i = q * NT + threadIdx.x;
        c[q] = i < n_blocks * K ? Pair{w.key[i], w.idx[i]} : Pair{kNone, kNone};
    }
    uint64_t pc[kSelBlocks / NT];
#pragma unroll
    for (uint32_t q = 0; q < kSelBlocks / NT; ++q) {
        const uint32_t i = q * NT + threadIdx.x;
        pc[q] = i < n_blocks ? w.cnt[i] : 0;
    }
    TopList<K> l;
    l.init();
    uint64_t cnt = 0;
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) l.insert(c[q]);
#pragma unroll
    for (uint32_t q = 0; q < kSelBlocks / NT; ++q) cnt += pc[q];
    for (int off = kWave / 2; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, kWave);
    if (threadIdx.x % kWave == 0) s_cnt[threadIdx.x / kWave] = cnt;
    block_topk<K, kNW>(l, s_pairs, [&](int r, const Pair &p) {
        if ((uint32_t)r < k) {
            out_idx[r] = p.idx;
            out_val[r] = p.idx == kNone ? INFINITY : value_of(p.key);
        }
    });
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int wv = 0; wv < kNW; ++wv) t += s_cnt[wv];
        out_cnt[0] = t;
    }
}

template <int K>
__global__ __launch_bounds__(kMergeThreads) void topk_merge_kernel(Top1Ws w, uint32_t n_blocks, uint32_t k,
                                                                   uint64_t *out_idx, double *out_val, uint64_t *out_cnt) {
    topk_merge_body<K, kMergeThreads>(w, n_blocks, k, out_idx, out_val, out_cnt);
}


// ------------------------------------------------------- top-k, with groups

// Workspace of a grouped top-k, three u64 per group and block of kSelBlocks: counts [group][block], keys and rows
// [group][block][k].
struct GroupWs {
    uint64_t *cnt, *key;
    uint32_t *row;
};
size_t topk_ws_bytes(uint32_t G) { return sizeof(uint64_t) * (2 * GUIDE_MAX_GROUPS + 3 * (size_t)kSelBlocks * G); }
GroupWs group_ws(void *ws, uint32_t G, uint32_t k, uint32_t n_blocks) {
    GroupWs w;
    w.cnt = (uint64_t *)ws;
    w.key = w.cnt + (size_t)G * n_blocks;
    w.row = (uint32_t *)(w.key + (size_t)G * n_blocks * k);
    return w;
}
constexpr uint32_t kGroupChunk = 4096;            // rows of a block's batch
// Blocks of the grouped pass: two per compute unit, fewer when the partials of more would not fit the workspace
// (8 + 12 k bytes per group and block: 512 blocks up to k = 3, 236 for k = 8; k = 1: the 1024 of blocks_for).
uint32_t group_blocks(uint64_t n, uint32_t k) {
    const uint64_t fit = 3 * sizeof(uint64_t) * kSelBlocks / (8 + 12 * (uint64_t)k), cap = 2 * (uint64_t)device_cus();
    uint64_t need = (n + kGroupChunk - 1) / kGroupChunk;
    need = need ? need : 1;
    need = need < cap ? need : cap;
    return (uint32_t)(need < fit ? need : fit);
}

// Counts a row of group g in every lane that is ok.  One lane does it where the rows of a wave are all of one group: 64
// atomics on one word take 64 turns (1.9 million rows of one group: 15.5 instead of 20 us).  Every lane of the wave must call.
__device__ inline void count_rows(uint32_t *s_cnt, uint32_t g, bool ok) {
    const uint64_t oks = __ballot(ok);
    if (oks == 0) return;
    const int lead = __ffsll((long long)oks) - 1;
    const uint32_t g0 = (uint32_t)__builtin_amdgcn_readlane((int)g, lead);
    if (__ballot(ok && g != g0) == 0) {
        if ((int)(threadIdx.x % kWave) == lead) atomicAdd(&s_cnt[g0], (uint32_t)__popcll(oks));
    } else if (ok) {
        atomicAdd(&s_cnt[g], 1u);
    }
}

// k = 1: one pass in which the rows of a group meet in a slot per wave and group (slot_update), whatever their order.  The
// lists below need a start and a merge inside the block, which one row per group does not pay for: 5000 rows of
// ten groups 6.0 us and 8 million falling rows of five groups 34 us like this, 9.5 - 12.5 us and 432 us with lists of one.
template <uint32_t MAXC>
__global__ __launch_bounds__(kBlock) void topk_group_first_kernel(const double *__restrict__ obj, RowFilter f,
                                                                  const uint32_t *__restrict__ group, uint32_t G, uint32_t n,
                                                                  GroupWs w) {
    __shared__ uint64_t s_key[kWaves][GUIDE_MAX_GROUPS], s_idx[kWaves][GUIDE_MAX_GROUPS];
    __shared__ uint32_t s_cnt[kWaves][GUIDE_MAX_GROUPS];
    const int wave = threadIdx.x / kWave;
    for (uint32_t i = threadIdx.x; i < kWaves * GUIDE_MAX_GROUPS; i += kBlock) {
        (&s_key[0][0])[i] = kNone;
        (&s_idx[0][0])[i] = kNone;
        (&s_cnt[0][0])[i] = 0;
    }
    __syncthreads();
    constexpr uint32_t U = 4;                                   // rows per thread in flight
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t base = (uint64_t)blockIdx.x * kBlock; base < n; base += U * stride) {       // block-uniform trip count
        RawRow<MAXC> raw[U];
        uint32_t grp[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint64_t at = base + u * stride + threadIdx.x;
            const uint32_t i = at < n ? (uint32_t)at : n;       // n: not there
            raw[u] = load_raw<false, MAXC>(obj, nullptr, f, i, n);
            grp[u] = group[i < n ? i : 0u];
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (base + u * stride >= n) break;                  // (uniform)
            const Row r = row_of<false, MAXC>(raw[u], f);
            const bool ok = r.pass && grp[u] < G;
            count_rows(s_cnt[wave], grp[u], ok);
            slot_update(s_key[wave], s_idx[wave], grp[u], ok, Pair{key_of(r.x), base + u * stride + threadIdx.x});
        }
    }
    __syncthreads();
    for (uint32_t g = threadIdx.x; g < G; g += kBlock) {
        Pair b = {s_key[0][g], s_idx[0][g]};
        uint64_t c = s_cnt[0][g];
        for (int wv = 1; wv < kWaves; ++wv) {
            b = pair_min(b, Pair{s_key[wv][g], s_idx[wv][g]});
            c += s_cnt[wv][g];
        }
        const size_t to = (size_t)g * gridDim.x + blockIdx.x;
        w.key[to] = b.key;
        w.row[to] = (uint32_t)b.idx;
        w.cnt[to] = c;
    }
}

constexpr uint32_t kGroupThreads = 1024;
constexpr uint32_t kGroupParts = 16;                       // parts of a batch whose least rows tighten the bounds; >= k
constexpr uint32_t kGroupSlots = 32;                       // rows of one group that a block holds at a time; > k
static_assert(kGroupParts >= GUIDE_MAX_TOPK && kGroupSlots >= 2 * GUIDE_MAX_TOPK, "a list of k rows must fit");
struct GroupLds {           // 596 bytes per group
    uint64_t *bound_key, *part_key, *slot_key;             // [G], [G][kGroupParts], [G][kGroupSlots]
    uint32_t *bound_row, *part_row, *slot_row, *n, *cnt;   // the same, rows in the slots, passing rows
};
constexpr size_t kGroupLdsBytes = sizeof(uint64_t) * (1 + kGroupParts + kGroupSlots) + sizeof(uint32_t) * (3 + kGroupParts + kGroupSlots);
static_assert(kGroupLdsBytes * GUIDE_MAX_GROUPS <= 65536, "the tables of a block fit the default LDS limit");

// Keeps the k least rows of every group's slots, in order, and lowers the bounds to the k-th of them.  To be called by the
// whole block; ends with a barrier.
__device__ inline void group_compact(const GroupLds &L, uint32_t G, uint32_t k) {
    constexpr uint32_t kPer = GUIDE_MAX_GROUPS * kGroupSlots / kGroupThreads;
    uint64_t key[kPer];
    uint32_t row[kPer], rank[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        const uint32_t i = q * kGroupThreads + threadIdx.x, g = i / kGroupSlots, at = i % kGroupSlots;
        rank[q] = kGroupSlots;                              // not there
        if (g < G) {
            const uint32_t n = L.n[g] < kGroupSlots ? L.n[g] : kGroupSlots;
            if (at < n) {
                key[q] = L.slot_key[i];
                row[q] = L.slot_row[i];
                rank[q] = 0;
#pragma unroll 2
                for (uint32_t j = 0; j < n; ++j) {
                    const uint64_t o = L.slot_key[g * kGroupSlots + j];
                    rank[q] += (o < key[q] || (o == key[q] && L.slot_row[g * kGroupSlots + j] < row[q])) ? 1u : 0u;
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        const uint32_t i = q * kGroupThreads + threadIdx.x, g = i / kGroupSlots;
        if (rank[q] < k) {
            L.slot_key[g * kGroupSlots + rank[q]] = key[q];
            L.slot_row[g * kGroupSlots + rank[q]] = row[q];
            if (rank[q] == k - 1 && (key[q] < L.bound_key[g] || (key[q] == L.bound_key[g] && row[q] < L.bound_row[g]))) {
                L.bound_key[g] = key[q];
                L.bound_row[g] = row[q];
            }
        }
        if (g < G && i % kGroupSlots == 0) L.n[g] = L.n[g] < k ? L.n[g] : k;
    }
    __syncthreads();
}

// One pass over the rows for any number of groups and k >= 2.  The block keeps, per group, up to kGroupSlots rows in LDS and
// a bound (key, row) with at least k of its rows at or below it.  Rows above the bound of their group, nearly all,
// cost a compare; the others are appended, all lanes side by side, and when a group's slots are full the k least of
// them stay.  A batch in which many rows are below their bounds (the first one; columns that fall with the row number;
// long runs of equal values) tightens the bounds first: the least row of each of sixteen parts of the batch per group,
// the k-th of which has k rows at or below it.  So no order of the rows makes a block append much more than k
// rows per group and batch.
// Bound by latency at this size (one batch per block): 1.9 million rows, ten groups, k = 3 and one constraint (40 MB) take
// 16.3 us + 5.6 us for the merge; k rounds over all rows 56 us a call.  8 million rows of 64 groups, k = 8: 81 us in random order, 108 us
// falling, 47 us all equal (k rounds: 336 us); one list per wave and group, whose rows enter one after the other: 263,
// 1210 and 200 us.  Blocks of 512 threads with eight rows each: 57 instead of 47 us (8 million rows, 64 groups, k = 3);
// the next batch under way meanwhile: 74 us (four rows, one block per compute unit then).
template <uint32_t MAXC>
__global__ __launch_bounds__(kGroupThreads, 8) void topk_group_kernel(const double *__restrict__ obj, RowFilter f,
                                                            const uint32_t *__restrict__ group, uint32_t G, uint32_t k,
                                                            uint32_t n, GroupWs w) {
    extern __shared__ __align__(16) unsigned char s_group[];
    __shared__ uint32_t s_any[3];
    uint32_t turn = 0;
    // true in every thread when any brings true; a barrier.  (Three flags in turn: the one that is cleared after a barrier
    // was read before it by all, and is written again after the next.)
    auto block_any = [&](bool mine) {
        if (mine) s_any[turn] = 1;
        __syncthreads();
        const bool any = s_any[turn] != 0;
        const uint32_t last = turn == 0 ? 2u : turn - 1;
        if (threadIdx.x == 0) s_any[last] = 0;
        turn = turn == 2 ? 0u : turn + 1;
        return any;
    };
    if (threadIdx.x < 3) s_any[threadIdx.x] = 0;
    GroupLds L;
    L.bound_key = (uint64_t *)s_group;
    L.part_key = L.bound_key + G;
    L.slot_key = L.part_key + G * kGroupParts;
    L.bound_row = (uint32_t *)(L.slot_key + G * kGroupSlots);
    L.part_row = L.bound_row + G;
    L.slot_row = L.part_row + G * kGroupParts;
    L.n = L.slot_row + G * kGroupSlots;
    L.cnt = L.n + G;
    for (uint32_t i = threadIdx.x; i < G; i += kGroupThreads) {
        L.bound_key[i] = kNone;
        L.bound_row[i] = ~0u;
        L.n[i] = 0;
        L.cnt[i] = 0;
    }
    auto clear_parts = [&]() {
        for (uint32_t i = threadIdx.x; i < G * kGroupParts; i += kGroupThreads) {
            L.part_key[i] = kNone;
            L.part_row[i] = ~0u;
        }
    };
    clear_parts();
    __syncthreads();
    constexpr uint32_t U = 4;
    ChunkWalk<U * kGroupThreads / kBlock> cw(kGroupChunk, n, gridDim.x);     // batches of kGroupThreads * U rows
    RawRow<MAXC> raw[U];
    uint32_t raw_g[U];
    auto request = [&]() {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = (uint32_t)cw.base + threadIdx.x + u * kGroupThreads;
            raw[u] = load_raw<false, MAXC>(obj, nullptr, f, i, (uint32_t)cw.end);
            raw_g[u] = group[i < (uint32_t)cw.end ? i : 0];
        }
    };
    bool first = true;                                          // no bounds yet
    while (cw.live()) {                                         // block-uniform trip count
        request();
        const uint32_t base = (uint32_t)cw.base + threadIdx.x;
        uint64_t key[U];
        uint32_t grp[U], in = 0;                                // in: bit u = row u may still be among the k least
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const Row r = row_of<false, MAXC>(raw[u], f);
            const bool ok = r.pass && raw_g[u] < G;
            grp[u] = ok ? raw_g[u] : 0u;
            key[u] = key_of(r.x);
            in |= ok ? 1u << u : 0u;
            count_rows(L.cnt, grp[u], ok);
        }
        cw.next();
        auto drop = [&]() {                                     // rows above their bounds; how many of the wave's are left
            uint32_t left = 0;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint64_t b = L.bound_key[grp[u]];
                const bool keep = ((in >> u) & 1u) && (key[u] < b || (key[u] == b && base + u * kGroupThreads <= L.bound_row[grp[u]]));
                in = keep ? in : in & ~(1u << u);
                left += (uint32_t)__popcll(__ballot(keep));
            }
            return left;
        };
        constexpr uint32_t kMany = kWave / 4;
        if (first || block_any(drop() > kMany)) {
            first = false;
            // (clear_parts() has run since the last time, and a barrier)
            auto part_of = [&](uint32_t u) {                    // scattered, so that no period of the rows lines up with it
                return grp[u] * kGroupParts + (((base + u * kGroupThreads) * 2654435761u) >> 28);
            };
            static_assert(kGroupParts == 16, "four bits of the product");
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if ((in >> u) & 1u) atomicMin((unsigned long long *)&L.part_key[part_of(u)], (unsigned long long)key[u]);
            __syncthreads();
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (((in >> u) & 1u) && L.part_key[part_of(u)] == key[u]) atomicMin(&L.part_row[part_of(u)], base + u * kGroupThreads);
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < G * kGroupParts; i += kGroupThreads) {
                const uint32_t g = i / kGroupParts, row = L.part_row[i];
                const uint64_t pk = L.part_key[i];
                uint32_t rank = 0;
#pragma unroll 4
                for (uint32_t j = 0; j < kGroupParts; ++j) {
                    const uint64_t o = L.part_key[g * kGroupParts + j];
                    rank += (o < pk || (o == pk && L.part_row[g * kGroupParts + j] < row)) ? 1u : 0u;
                }
                // (rows in the parts are at or below the old bound, so this one is not above it)
                if (rank == k - 1 && pk != kNone) {
                    L.bound_key[g] = pk;
                    L.bound_row[g] = row;
                }
            }
            __syncthreads();
            clear_parts();
            drop();
        }
        for (;;) {
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                if (!((in >> u) & 1u)) continue;
                const uint32_t at = atomicAdd(&L.n[grp[u]], 1u);
                if (at < kGroupSlots) {
                    L.slot_key[grp[u] * kGroupSlots + at] = key[u];
                    L.slot_row[grp[u] * kGroupSlots + at] = base + u * kGroupThreads;
                    in &= ~(1u << u);
                }
            }
            // full slots: at least kGroupSlots - k of the rows left are done with in the next turn
            if (!block_any(in != 0)) break;
            group_compact(L, G, k);
            drop();
        }
    }
    group_compact(L, G, k);
    for (uint32_t i = threadIdx.x; i < G * k; i += kGroupThreads) {
        const uint32_t g = i / k, j = i - g * k;
        const size_t to = ((size_t)g * gridDim.x + blockIdx.x) * k;
        const bool there = j < L.n[g];
        w.key[to + j] = there ? L.slot_key[g * kGroupSlots + j] : kNone;
        w.row[to + j] = there ? L.slot_row[g * kGroupSlots + j] : ~0u;
    }
    for (uint32_t g = threadIdx.x; g < G; g += kGroupThreads) w.cnt[(size_t)g * gridDim.x + blockIdx.x] = L.cnt[g];
}

// One block per group: the k least of the block partials, and the count.  K >= k: places of the threads' lists.
template <int K>
__global__ __launch_bounds__(kBlock) void topk_group_merge_kernel(GroupWs w, uint32_t n_blocks, uint32_t k, uint64_t *out_idx,
                                                                  double *out_val, uint64_t *out_cnt) {
    __shared__ Pair s_pairs[kWaves][K];
    __shared__ uint64_t s_cnt[kWaves];
    const uint32_t g = blockIdx.x;
    const uint64_t *key = w.key + (size_t)g * n_blocks * k;
    const uint32_t *row = w.row + (size_t)g * n_blocks * k;
    TopList<K> l;
    l.init();
    uint64_t cnt = 0;
    const uint32_t total = n_blocks * k;
    for (uint32_t i0 = threadIdx.x; i0 < total; i0 += 4 * kBlock) {             // four loads in flight
        uint64_t c[4];
        uint32_t c_row[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {
            const uint32_t i = i0 + u * kBlock;
            c[u] = i < total ? key[i] : kNone;
            c_row[u] = i < total ? row[i] : ~0u;
        }
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
            if (c_row[u] != ~0u) l.insert(Pair{c[u], (uint64_t)c_row[u]});
    }
    for (uint32_t i = threadIdx.x; i < n_blocks; i += kBlock) cnt += w.cnt[(size_t)g * n_blocks + i];
    for (int off = kWave / 2; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, kWave);
    if (threadIdx.x % kWave == 0) s_cnt[threadIdx.x / kWave] = cnt;
    block_topk<K, kWaves>(l, s_pairs, [&](int r, const Pair &p) {
        if ((uint32_t)r < k) {
            out_idx[(size_t)g * k + r] = p.idx;
            out_val[(size_t)g * k + r] = p.idx == kNone ? INFINITY : value_of(p.key);
        }
    });
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int wv = 0; wv < kWaves; ++wv) t += s_cnt[wv];
        out_cnt[g] = t;
    }
}

// --------------------------------------------------------------------- Pareto
//
// Three launches.  The first can ride along with a top-k pass or with the kernel that produces the
// columns; a top-k over the same columns can ride along with the second, and a top-k merge with the last.
// Sample: kSampleBlocks blocks take a scattered sample of rows.  It fixes the stretch of x that the bins
// slice (kBins equal slices of key space, clamped at both ends, so a lower bin means a strictly smaller x),
// and every block hands over rows of the front of its sample: evenly spaced ones where they are stored columns
// (pareto_prepare_body), the rightmost of each wave where the evaluation kernel's extra blocks work them out (store_sample_front).
// The block that takes sample 0 also resets the counters that the next two kernels accumulate into.
// Filter: every block bins the handed-over sample rows (least y per bin, exclusive prefix-min) and keeps a
// row when no sample row of a strictly lower bin has a y at or below its own.  The kept rows contain the
// front, and every other kept row is dominated by a kept one.  Kept rows are appended as (row, keys).
// Finish: kept rows are binned; those that a kept row of a strictly lower bin dominates (least y per bin
// over the kept rows, exclusive prefix-min) or that their own bin's representative dominates are dropped,
// the rest are grouped by bin and tested exactly inside their bin (or sorted, where they crowd), and front members are written at
// (front members of lower bins) + (rank inside the bin), which orders the output by (x, y, row).  One block does
// this in LDS for up to kStage kept rows; more are shared out among kLargeParts blocks by runs of bins, each of which does the
// same with what is left of its share, in bins of its own, bins of bins, and rounds.

// Sample rows per thread of the row sample's blocks, and the row that sample number k stands for (n: none): all of them when the
// sample is larger than the selection, otherwise one at a scrambled place in each of as many stretches, so that no period of
// the rows' layout lines up with the sample.  Four rows a thread halve what the filter pass keeps, but 64 compute units take
// 4 us longer to fetch four columns' worth of scattered lines.  In us a call with one / four, a uniform cloud, a band along the
// diagonal, a thin front: 400 000 rows 20.7 / 22.6, 41 / 43, 87 / 83; 1.2 million 24.7 / 25.6, 59 / 59, 182 / 158; 1.5 million
// 26.7 / 25.7, 66 / 64, 216 / 187; 1.9 million 29.4 / 27.7, 71 / 71, 261 / 231; 4 million 40 / 32, 117 / 107, 504 / 449;
// 16 million 91 / 68, 364 / 318, 1917 / 1597.
constexpr uint32_t kSampleDeep = 4, kDeepSampleRows = 1500000;
__device__ inline uint32_t sample_deep(uint32_t n) { return n > kDeepSampleRows ? kSampleDeep : 1u; }
__device__ inline uint32_t sample_of(uint32_t k, uint32_t n) {
    const uint32_t total = kSampleBlocks * kBlock * sample_deep(n);
    if (n <= total) return k < n ? k : n;
    const uint32_t stride = n / total, rest = n - stride * total;           // stretches of stride or stride + 1 rows
    return k * stride + (uint32_t)((uint64_t)k * rest / total) + ((k * 2654435761u) >> 8) % stride;
}

constexpr uint32_t kStage = 4096;        // survivors whose records the finishing block holds in LDS
constexpr uint32_t kFinishThreads = 1024;

// Caller workspace of the Pareto path (kParetoRowBytes a row).
struct ParetoWs {
    uint64_t *skx, *sky;  // [n]: keys of surviving rows
    uint32_t *surv;       // [n]: surviving rows, arbitrary order
    // large-front path only:
    uint32_t *staged;     // [n]: per part of the front, from its first survivor slot on: positions of its survivors, then its front
                          // members' rows in order
    uint32_t *grouped;    // [n]: positions into surv, grouped by bin (parts whose survivors do not fit LDS)
};
size_t pareto_ws_bytes(uint64_t n) { return (size_t)n * kParetoRowBytes + 256; }
ParetoWs pareto_ws(void *ws, uint64_t n) {
    ParetoWs w;
    w.skx = (uint64_t *)ws;
    w.sky = w.skx + n;
    w.surv = (uint32_t *)(w.sky + n);
    w.staged = w.surv + n;
    w.grouped = w.staged + n;
    return w;
}

struct Binning {
    uint64_t lo;
    uint32_t shift;
    __device__ uint32_t operator()(uint64_t kx) const {
        if (kx <= lo) return 0;
        const uint64_t b = (kx - lo) >> shift;
        return b < kBins ? (uint32_t)b : kBins - 1;
    }
};
__device__ inline Binning binning_of(uint64_t lo, uint64_t hi) {
    Binning b;
    b.lo = lo;
    const uint64_t span = hi - lo;
    // least shift with (span >> shift) < kBins
    const uint32_t bits = span ? 64u - (uint32_t)__builtin_clzll(span) : 0u;   // span < 2^bits
    constexpr uint32_t kBinBits = 12;
    static_assert((1u << kBinBits) == kBins, "kBins is a power of two");
    b.shift = bits > kBinBits ? bits - kBinBits : 0u;
    return b;
}
// The stretch of keys up to `hi` that bins b_lo .. b_hi slice (hi: the end of the binning's range, beyond which only a few rows are;
// what is below the range is in its first bin).
struct Stretch {
    uint64_t lo, hi;
};
__device__ inline Stretch stretch_of(const Binning &bin, uint64_t hi, uint32_t b_lo, uint32_t b_hi) {
    const uint64_t lo = bin.lo + ((uint64_t)b_lo << bin.shift), end = bin.lo + (((uint64_t)b_hi + 1) << bin.shift) - 1;
    return Stretch{lo, end < lo ? hi : min_u64(end, hi)};           // (end < lo: it is beyond 64 bits)
}

// kBins-entry tables in LDS that a block scans are stored with one unused slot after every PER
// entries (PER = entries per thread of the scan): thread t's entries then start at slot t * (PER + 1),
// and the lanes of a wave reach different banks when each reads its own j-th entry.
template <uint32_t PER>
__device__ inline uint32_t padded(uint32_t i) { return i + i / PER; }
template <uint32_t PER>
constexpr uint32_t padded_size() { return kBins + kBins / PER + 1; }
constexpr uint32_t kPerPass = kBins / kBlock;             // table entries per thread of a streaming block
constexpr uint32_t kPerFinish = kBins / 1024;             // ... of the finishing block

// Thread t of the NT-thread block owns the `per` consecutive entries v[] of a
// table; returns the minimum over all entries before its first one
// (scan in the wave, wave totals through LDS; one block barrier).
// s_tmp: NT / kWave entries.
template <uint32_t NT, uint32_t per>
__device__ inline uint64_t prefix_min_before(const uint64_t (&v)[per], uint64_t *s_tmp) {
    constexpr uint32_t nw = NT / kWave;
    const uint32_t t = threadIdx.x, lane = t % kWave, wave = wave_number();
    uint64_t m = kNone;
#pragma unroll
    for (uint32_t j = 0; j < per; ++j) m = min_u64(m, v[j]);
    const uint64_t inc = wave_scan_min(m);              // inclusive scan of thread minima in the wave
    if (lane == kWave - 1) s_tmp[wave] = inc;
    uint64_t run = __shfl_up(inc, 1, kWave);            // exclusive within the wave
    if (lane == 0) run = kNone;
    __syncthreads();
    return min_u64(run, min_before_wave<nw>(s_tmp, wave));
}

// Range that the bins slice, from a scattered sample of rows: low end = least x of
// passing sample rows, high end = x of the sample row with the least y (rows
// beyond it are dominated by that row unless their y is smaller still; they share
// the last bin).  Any monotone binning is correct -- the sample only decides how
// finely the interesting stretch of x is resolved.
// A block bins its sample rows over its own range (least y per bin, exclusive prefix-min) and
// hands over the row of every bin whose least y is below that of all lower bins; of more than kSampleFrontPer such
// rows, evenly spaced ones, so that every stretch of x gets its share.  Any subset of rows is valid, but what is not handed
// over prunes nothing: 1.9 million rows whose front has 8000 (4000 and 2800) members keep 40 000 (8600) of them like this, and
// kept 419 000 (18 300) with 256 rows a block of which each wave handed over its eight rightmost.  11 us (7 us).
constexpr uint32_t kSampleBins = 1024;                    // of a sampling block
__device__ void pareto_prepare_body(uint32_t block, const double *__restrict__ x, const double *__restrict__ y,
                                    const RowFilter &f, uint32_t n, SelectScratch *sc) {
    constexpr uint32_t NT = kBlock, R = kSampleDeep, P = kSampleBins / NT, NW = NT / kWave;
    constexpr uint8_t kNoSlot = 0xFF;
    static_assert(kSampleFrontPer < kNoSlot && kSampleFrontPer <= NT, "a slot number fits a byte, and a thread each");
    __shared__ uint64_t s_low[kSampleBins + kSampleBins / P], s_tmp[NW], s_lo[NW];
    __shared__ Pair s_best[NW];
    __shared__ uint8_t s_slot[kSampleBins];
    __shared__ uint32_t s_sum[NW];
    const uint32_t t = threadIdx.x, lane = t % kWave, wave = t / kWave, deep = sample_deep(n);
    if (block == 0 && t == 0) sc->counters[0] = sc->counters[1] = 0;        // neutral state for the kernels that follow
    RawRow<GUIDE_MAX_CONSTRAINTS> raw[R];
#pragma unroll
    for (uint32_t q = 0; q < R; ++q) {
        raw[q].valid = false;
        if (q < deep) raw[q] = load_raw<true, GUIDE_MAX_CONSTRAINTS>(x, y, f, sample_of((q * NT + t) * kSampleBlocks + block, n), n);
    }
    for (uint32_t i = t; i < kSampleBins + kSampleBins / P; i += NT) s_low[i] = kNone;
    uint64_t lo = kNone, kx[R], ky[R];
    bool pass[R];
    Pair best = {kNone, kNone};                                     // (y key, x key) of the least y
#pragma unroll
    for (uint32_t q = 0; q < R; ++q) {
        pass[q] = false;
        kx[q] = ky[q] = kNone;
        if (q >= deep) continue;                        // (uniform)
        const Row r = row_of<true, GUIDE_MAX_CONSTRAINTS>(raw[q], f);
        pass[q] = r.pass;
        kx[q] = pass[q] ? key_of(r.x) : kNone;
        ky[q] = pass[q] ? key_of(r.y) : kNone;
        lo = min_u64(lo, kx[q]);
        best = pair_min(best, Pair{ky[q], kx[q]});
    }
    lo = wave_min(lo);
    best = wave_min(best);
    if (lane == 0) {
        s_lo[wave] = lo;
        s_best[wave] = best;
    }
    __syncthreads();
    for (uint32_t w = 0; w < NW; ++w) {
        lo = min_u64(lo, s_lo[w]);
        best = pair_min(best, s_best[w]);
    }
    Pair *slots = sc->sample_front + block * kSampleFrontPer;
    if (t == 0) {
        sc->sample_lo[block] = lo;
        sc->sample_best[block] = best;
    }
    if (lo == kNone) {                                              // no sample row passes (block-uniform)
        if (t < kSampleFrontPer) slots[t] = Pair{kNone, kNone};
        return;
    }
    const Binning fine = binning_of(lo, best.idx);
    auto bin = [&](uint64_t k) { return fine(k) / (kBins / kSampleBins); };
#pragma unroll
    for (uint32_t q = 0; q < R; ++q)
        if (pass[q]) atomicMin((unsigned long long *)&s_low[padded<P>(bin(kx[q]))], (unsigned long long)ky[q]);
    __syncthreads();
    // corners: bins whose least y is below that of all lower bins, numbered from the left
    uint64_t v[P];
#pragma unroll
    for (uint32_t j = 0; j < P; ++j) v[j] = s_low[t * (P + 1) + j];
    uint64_t run = prefix_min_before<NT, P>(v, s_tmp);
    uint32_t corners = 0;                                           // bit j: entry j is one
#pragma unroll
    for (uint32_t j = 0; j < P; ++j) {
        corners |= v[j] < run ? 1u << j : 0u;
        run = min_u64(run, v[j]);
    }
    const uint32_t mine = (uint32_t)__popc(corners), incl = wave_scan_sum(mine);
    if (lane == kWave - 1) s_sum[wave] = incl;
    __syncthreads();
    uint32_t at = incl - mine, total = 0;
    for (uint32_t w = 0; w < NW; ++w) {
        at += w < wave ? s_sum[w] : 0u;
        total += s_sum[w];
    }
    const uint32_t per = total < kSampleFrontPer ? total : kSampleFrontPer;     // corner r goes to slot r * per / total, the last one that would
#pragma unroll
    for (uint32_t j = 0; j < P; ++j) {
        uint32_t slot = kNoSlot;
        if ((corners >> j) & 1u) {
            const uint32_t s0 = at * per / total, s1 = (at + 1) * per / total;
            slot = s0 != s1 ? s0 : kNoSlot;
            ++at;
        }
        s_slot[t * P + j] = (uint8_t)slot;
    }
    if (t < kSampleFrontPer && t >= per) slots[t] = Pair{kNone, kNone};
    __syncthreads();
    // (rows that tie in y inside a bin write one after the other, each a valid one: 16 bytes by one store)
#pragma unroll
    for (uint32_t q = 0; q < R; ++q) {
        const uint32_t b = pass[q] ? bin(kx[q]) : 0u;
        if (pass[q] && s_slot[b] != kNoSlot && s_low[padded<P>(b)] == ky[q]) slots[s_slot[b]] = Pair{ky[q], kx[q]};
    }
}
__global__ __launch_bounds__(kBlock) void pareto_prepare_kernel(const double *__restrict__ x,
                                                                const double *__restrict__ y, RowFilter f, uint32_t n,
                                                                SelectScratch *sc) {
    pareto_prepare_body(blockIdx.x, x, y, f, n, sc);
}

// Combines the kSampleBlocks per-block sample partials (the same result in every block): the
// first wave loads them, one per lane, and reduces; s_rng (2 entries) carries the result to
// the other waves.  Contains a block barrier.
__device__ inline Binning sampled_binning(const SelectScratch *sc, uint64_t *s_rng) {
    static_assert(kSampleBlocks == kWave, "one partial per lane of the first wave");
    if (threadIdx.x < kWave) {
        uint64_t lo = wave_min(sc->sample_lo[threadIdx.x]);
        const Pair best = wave_min(sc->sample_best[threadIdx.x]);
        uint64_t hi = best.idx;
        if (lo == kNone || hi < lo) {   // no passing sample row: one slice per 2^52 keys
            lo = 0;
            hi = kNone;
        }
        if (threadIdx.x == 0) {
            s_rng[0] = lo;
            s_rng[1] = hi;
        }
    }
    __syncthreads();
    return binning_of(s_rng[0], s_rng[1]);
}

// Exclusive prefix-min over a (padded) kBins-entry table in LDS, in place, by the NT threads of the block.
template <uint32_t NT>
__device__ inline void scan_min_excl(uint64_t *s_io, uint64_t *s_tmp) {
    constexpr uint32_t per = kBins / NT;
    const uint32_t t = threadIdx.x;
    uint64_t v[per];
#pragma unroll
    for (uint32_t j = 0; j < per; ++j) v[j] = s_io[t * (per + 1) + j];
    uint64_t run = prefix_min_before<NT, per>(v, s_tmp);
#pragma unroll
    for (uint32_t j = 0; j < per; ++j) {
        s_io[t * (per + 1) + j] = run;
        run = min_u64(run, v[j]);
    }
    __syncthreads();
}

// Exclusive prefix-sum over a kBins-entry table, in place, by the NT threads of the block; the total
// goes to entry kBins.  PAD: the table is a padded LDS table; otherwise plain (global memory).
// s_tmp: NT / kWave entries.
template <uint32_t NT, bool PAD>
__device__ inline void scan_sum_excl(uint32_t *io, uint32_t *s_tmp) {
    constexpr uint32_t per = kBins / NT, nw = NT / kWave, pitch = PAD ? per + 1 : per;
    const uint32_t t = threadIdx.x, lane = t % kWave, wave = wave_number();
    uint32_t v[per], m = 0;
#pragma unroll
    for (uint32_t j = 0; j < per; ++j) {
        v[j] = io[t * pitch + j];
        m += v[j];
    }
    const uint32_t inc = wave_scan_sum(m);
    if (lane == kWave - 1) s_tmp[wave] = inc;
    __syncthreads();
    uint32_t total;
    uint32_t run = inc - m + sum_before_wave<nw>(s_tmp, wave, total);
#pragma unroll
    for (uint32_t j = 0; j < per; ++j) {
        io[t * pitch + j] = run;
        run += v[j];
    }
    if (t == 0) io[PAD ? padded<per>(kBins) : kBins] = total;
    __syncthreads();
}

// A top-k selection over the same rows that reads nothing but the Pareto selection's two columns and its
// flag column: the filter pass has those values in registers anyway and keeps the per-lane lists
// beside its own work, so the top-k needs no pass of its own.
struct SharedTopk {
    uint32_t obj_is_y;             // objective: 0 = the x column, 1 = the y column
    uint32_t use_feasible;         // rows with flag 0 do not pass
    uint32_t n_con;                // <= 2 constraints, each on x or y
    uint32_t con_is_y[2];
    double cap[2];
    Top1Ws w;                      // block partials, as written by the top-k pass
};

// The filter pass of the three-launch form: the sampling blocks have handed over the front of their sample
// rows (SelectScratch::sample_front); every block bins those few rows in LDS (least y per bin, then its
// exclusive prefix-min) and keeps a row when no sample row of a strictly lower bin has a y at or below its
// own.  Every row of the front is kept, and every other kept row is dominated by a kept one (its
// dominators are themselves dominated by a front row, and domination is transitive).  Kept rows are appended
// as (row, keys); the finishing kernel makes the bins' tables from them.
// KT: pairs per block partial of a top-k that shares the columns (0 = none).
template <uint32_t MAXC, int KT, uint32_t U>
__global__ __launch_bounds__(kBlock) void pareto_filter_kernel(const double *__restrict__ x, const double *__restrict__ y,
                                                               RowFilter f, uint32_t n, ParetoWs w, SelectScratch *sc,
                                                               SharedTopk topk, uint32_t chunk) {
    __shared__ uint64_t s_lower[padded_size<kPerPass>()], s_tmp[kWaves], s_rng[2];
    constexpr int KL = KT ? KT : 1;
    constexpr uint32_t kPerSample = kSampleBlocks * kSampleFrontPer / kBlock;
    static_assert(kSampleBlocks * kSampleFrontPer % kBlock == 0, "whole sample rows per thread");
    const int lane = threadIdx.x % kWave;
    TopList<KL> list;
    uint32_t n_pass = 0;                                // rows of one lane: fewer than 2^32
    if (KT) list.init();
    // requested first, and in this order: the sample rows, then the first batch of rows, whose latency
    // overlaps the set-up of the table
    Pair sf[kPerSample];
#pragma unroll
    for (uint32_t j = 0; j < kPerSample; ++j) sf[j] = sc->sample_front[j * kBlock + threadIdx.x];
    RawRow<MAXC> r[U];
    ChunkWalk<U> cw(chunk, n, gridDim.x);
    if (cw.live()) {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            r[u] = load_raw<true, MAXC>(x, y, f, (uint32_t)cw.base + threadIdx.x + u * kBlock, (uint32_t)cw.end);
    }
    for (uint32_t i = threadIdx.x; i < padded_size<kPerPass>(); i += kBlock) s_lower[i] = kNone;
    const Binning bin = sampled_binning(sc, s_rng);     // its barrier also covers the table above
#pragma unroll
    for (uint32_t j = 0; j < kPerSample; ++j)
        if (sf[j].idx != kNone)
            atomicMin((unsigned long long *)&s_lower[padded<kPerPass>(bin(sf[j].idx))], (unsigned long long)sf[j].key);
    __syncthreads();
    scan_min_excl<kBlock>(s_lower, s_tmp);              // least y of the sample rows in strictly lower bins
    // Kept rows are appended once per block and batch: the counts of the waves meet in LDS (alternating tables: a wave may count
    // the next batch while another still reads this one), one thread takes room for all.  An atomic per wave, on one counter, is a
    // queue of 3700 where kept rows are spread over the columns: 1.9 million rows took 38 us that way, 18 300 kept.
    __shared__ uint32_t s_kept[2][kWaves], s_at;
    uint32_t turn = 0;
    // block-uniform trip count: the ballots and barriers below need every lane
    while (cw.live()) {
        const uint32_t base = (uint32_t)cw.base;
        // the next batch is requested before this one is worked on
        RawRow<MAXC> rn[U];
        cw.next();
        const bool more = cw.live();
        if (more) {
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                rn[u] = load_raw<true, MAXC>(x, y, f, (uint32_t)cw.base + threadIdx.x + u * kBlock, (uint32_t)cw.end);
        }
        uint32_t keep_bits = 0, total = 0, before[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const Row q = row_of<true, MAXC>(r[u], f);
            const bool keep = q.pass && key_of(q.y) < s_lower[padded<kPerPass>(bin(key_of(q.x)))];
            const uint64_t mask = __ballot(keep);
            before[u] = total + (uint32_t)__popcll(mask & ((1ull << lane) - 1));
            total += (uint32_t)__popcll(mask);
            keep_bits |= keep ? 1u << u : 0u;
        }
        if (lane == 0) s_kept[turn][threadIdx.x / kWave] = total;
        __syncthreads();
        uint32_t at = 0, block_total = 0;
#pragma unroll
        for (uint32_t wv = 0; wv < kWaves; ++wv) {
            at += wv < threadIdx.x / kWave ? s_kept[turn][wv] : 0u;
            block_total += s_kept[turn][wv];
        }
        turn ^= 1u;
        if (block_total) {                              // block-uniform
            if (threadIdx.x == 0) s_at = atomicAdd(&sc->counters[0], block_total);
            __syncthreads();
            at += s_at;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                if ((keep_bits >> u) & 1u) {
                    const Row q = row_of<true, MAXC>(r[u], f);
                    const uint64_t kx = key_of(q.x), ky = key_of(q.y);
                    const uint32_t slot = at + before[u];
                    w.surv[slot] = base + threadIdx.x + u * kBlock;
                    w.skx[slot] = kx;
                    w.sky[slot] = ky;
                }
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = base + threadIdx.x + u * kBlock;
            if (KT) {
                const double obj = topk.obj_is_y ? r[u].y : r[u].x;
                bool ok = r[u].valid && (!topk.use_feasible || r[u].fe != 0) && obj == obj;
#pragma unroll
                for (uint32_t c = 0; c < 2; ++c)
                    if (c < topk.n_con) ok = ok && ((topk.con_is_y[c] ? r[u].y : r[u].x) <= topk.cap[c]);
                if (ok) {
                    ++n_pass;
                    list.insert_ascending(Pair{key_of(obj), (uint64_t)i});
                }
            }
        }
        if (more) {
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) r[u] = rn[u];
        }
    }
    if (KT) {
        __shared__ Pair s_pairs[kWaves][KL];
        __shared__ uint64_t s_cnt[kWaves];
        int my_rank = -1;
        Pair my_pair = {kNone, kNone};
        const uint32_t wave_pass = wave_sum(n_pass);
        if (threadIdx.x % kWave == 0) s_cnt[threadIdx.x / kWave] = wave_pass;
        block_topk<KL, kWaves>(list, s_pairs, [&](int rk, const Pair &p) {
            my_rank = rk;
            my_pair = p;
        });                                             // (contains the barrier that publishes s_cnt)
        if (my_rank >= 0) {
            topk.w.key[(size_t)blockIdx.x * KL + my_rank] = my_pair.key;
            topk.w.idx[(size_t)blockIdx.x * KL + my_rank] = my_pair.idx;
        }
        if (threadIdx.x == 0) {
            uint64_t c = 0;
            for (int wv = 0; wv < kWaves; ++wv) c += s_cnt[wv];
            topk.w.cnt[blockIdx.x] = c;
        }
    }
}

// A value that is the same in all lanes of the wave, kept in scalar registers.
__device__ inline uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ inline uint64_t uniform(uint64_t v) { return (uint64_t)uniform((uint32_t)(v >> 32)) << 32 | uniform((uint32_t)v); }

// threadIdx.x, formed anew at every use: what follows from it is not kept in registers across the finishing kernel's rounds.
__device__ inline uint32_t thread_here() {
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    __builtin_assume(t < 1024);
    return t;
}

// Least and greatest x and least y of some records.
struct KeyRange {
    uint64_t lo, hi, y;
    static __device__ KeyRange none() { return KeyRange{kNone, 0, kNone}; }
    __device__ void add(uint64_t kx, uint64_t ky) {
        lo = min_u64(lo, kx);
        hi = hi < kx ? kx : hi;
        y = min_u64(y, ky);
    }
};

// LDS of the finishing kernel.
struct FinishLds {
    uint32_t off[padded_size<kPerFinish>()];    // first survivor slot per bin (exclusive scan of the bin counts)
    uint32_t foff[padded_size<kPerFinish>()];   // front members per bin, then their exclusive scan
    uint32_t cur[kBins];                        // fill level per bin while grouping; then the list of front members
    uint32_t tmp[kFinishThreads / kWave];
    uint64_t tmp64[kFinishThreads / kWave];
    union {
        struct {
            uint64_t kx[kStage], ky[kStage];    // staged survivor records, grouped by bin
            uint32_t row[kStage];
        };
        // before anything is staged: per bin, the least y among the survivors of strictly lower bins (padded table), and the
        // least x among its survivors with the bin's least y
        struct {
            uint64_t lower[padded_size<kPerFinish>()], rep[kBins];
        };
    };
    uint16_t bin[kStage];
    uint8_t flag[kStage];
    uint32_t nfront, first, last, alive, is_last, todo;
    uint32_t part_base[kWave], part_lo[kWave], part_cnt[kWave];
    uint64_t rng[2];
    KeyRange range[kFinishThreads / kWave];
};

// The front among `cnt` survivor records staged in LDS, grouped by bin: record i of bin b sits at
// L.off[b] + i.  L.foff must be zero and the staging complete (the function starts with a barrier).
// Calls emit(position, row) for every front member, position = its rank by (bin, x, y, row) among the
// front members staged here, and returns their number.
// GROUP lanes per survivor (8 or 1): they share out the members of its bin, four LDS reads in flight each, and
// meet through a wave ballot.  A survivor's test is a chain of dependent LDS reads, so many survivors are kept
// in flight.  Up to 1024 survivors, eight lanes each are fastest (one lane per survivor: one round over all of
// them but longer chains, +1 to +6 us, the fullest bin setting the pace); beyond, one lane each saves more
// rounds (a round over 128 survivors costs about as much as one over 1024) than the chains cost.
template <uint32_t GROUP, typename Emit>
__device__ inline uint32_t staged_front_by(FinishLds &L, uint32_t cnt, Emit &&emit) {
    constexpr uint32_t P = kPerFinish, group = GROUP, q_step = kFinishThreads / group;
    constexpr uint64_t group_mask = group < 64 ? (1ull << group) - 1 : ~0ull;
    const uint32_t t = thread_here(), lane = t % kWave, sub = lane % group, shift = lane - sub;
    __syncthreads();
    const uint32_t cnt_pad = (cnt + q_step - 1) / q_step * q_step;      // wave-uniform trip count for the ballot
    for (uint32_t q = t / group; q < cnt_pad; q += q_step) {
        const bool live = q < cnt;
        const uint64_t kx = live ? L.kx[q] : 0, ky = live ? L.ky[q] : 0;
        const uint32_t b = live ? L.bin[q] : 0;
        bool dom = false;
        const uint32_t beg = live ? L.off[padded<P>(b)] : 0, end = live ? L.off[padded<P>(b + 1)] : beg;
        for (uint32_t j = beg + sub; j < end; j += 4 * group) {
            uint64_t jx[4], jy[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {      // past the end: the bin's first member once more
                const uint32_t jj = j + u * group < end ? j + u * group : beg;
                jx[u] = L.kx[jj];
                jy[u] = L.ky[jj];
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u)
                dom = dom || (jx[u] <= kx && jy[u] <= ky && (jx[u] < kx || jy[u] < ky));
        }
        const bool dominated = ((__ballot(dom) >> shift) & group_mask) != 0;
        if (live && sub == 0) {
            L.flag[q] = dominated ? 0 : 1;
            if (!dominated) {
                atomicAdd(&L.foff[padded<P>(b)], 1u);
                L.cur[atomicAdd(&L.nfront, 1u)] = q;        // L.cur is free again: list of front members
            }
        }
    }
    __syncthreads();
    scan_sum_excl<kFinishThreads, true>(L.foff, L.tmp);
    const uint32_t nf = uniform(L.nfront);
    const uint32_t f_pad = (nf + q_step - 1) / q_step * q_step;          // wave-uniform trip count for the shuffles
    for (uint32_t qf = t / group; qf < f_pad; qf += q_step) {
        const bool live = qf < nf;
        const uint32_t q = live ? L.cur[qf] : 0;
        const uint64_t kx = live ? L.kx[q] : 0, ky = live ? L.ky[q] : 0;
        const uint32_t b = live ? L.bin[q] : 0, i = live ? L.row[q] : 0;
        const uint32_t beg = live ? L.off[padded<P>(b)] : 0, end = live ? L.off[padded<P>(b + 1)] : 0;
        uint32_t rank = 0;                          // front members of the bin that come before this one
        for (uint32_t j = beg + sub; j < end; j += 4 * group) {
            uint64_t jx[4], jy[4];
            uint32_t jr[4];
            bool on[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t jj = j + u * group;
                on[u] = jj < end;
                const uint32_t jc = on[u] ? jj : beg;
                on[u] = on[u] && L.flag[jc];
                jx[u] = L.kx[jc];
                jy[u] = L.ky[jc];
                jr[u] = L.row[jc];
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u)
                rank += (on[u] && (jx[u] < kx || (jx[u] == kx && (jy[u] < ky || (jy[u] == ky && jr[u] < i))))) ? 1u : 0u;
        }
        for (uint32_t off = 1; off < group; off <<= 1) rank += __shfl_xor(rank, off, kWave);
        if (live && sub == 0) emit(L.foff[padded<P>(b)] + rank, i);
    }
    return nf;
}

// The same by sorting: for records that crowd in few bins, whatever their values.  In the order of (x, y, row) a record is on
// the front when no pair (y, x) before it is less than its own (one with a lower y, or with the same y and a lower x).
template <typename Emit>
__device__ inline uint32_t sorted_front(FinishLds &L, uint32_t cnt, Emit &&emit) {
    constexpr uint32_t NT = kFinishThreads, PER = kStage / NT;
    const uint32_t t = thread_here(), lane = t % kWave, wave = t / kWave;
    uint32_t n = 2;                                     // records and padding (which sorts behind every record)
    while (n < cnt) n *= 2;
    __syncthreads();
    for (uint32_t i = cnt + t; i < n; i += NT) {
        L.kx[i] = L.ky[i] = kNone;
        L.row[i] = ~0u;
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t k = 2; k <= n; k *= 2) {
#pragma unroll 1
        for (uint32_t j = k / 2; j; j /= 2) {
#pragma unroll 1
            for (uint32_t p = t; p < n / 2; p += NT) {
                const uint32_t a = 2 * p - (p & (j - 1)), b = a + j;
                const uint64_t ax = L.kx[a], bx = L.kx[b], ay = L.ky[a], by = L.ky[b];
                const uint32_t ar = L.row[a], br = L.row[b];
                const bool after = ax > bx || (ax == bx && (ay > by || (ay == by && ar > br)));
                if (after == ((a & k) == 0)) {
                    L.kx[a] = bx; L.kx[b] = ax;
                    L.ky[a] = by; L.ky[b] = ay;
                    L.row[a] = br; L.row[b] = ar;
                }
            }
            __syncthreads();
        }
    }
    // thread t owns PER consecutive records: least pair before its first one, front members before them
    Pair v[PER], run = {kNone, kNone};
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const uint32_t i = t * PER + q;
        v[q] = i < cnt ? Pair{L.ky[i], L.kx[i]} : Pair{kNone, kNone};
        run = pair_min(run, v[q]);
    }
    for (uint32_t off = 1; off < kWave; off *= 2) {
        const Pair o = {__shfl_up(run.key, off, kWave), __shfl_up(run.idx, off, kWave)};
        if (lane >= off) run = pair_min(run, o);
    }
    if (lane == kWave - 1) L.range[wave].lo = run.key, L.range[wave].hi = run.idx;
    run = Pair{__shfl_up(run.key, 1, kWave), __shfl_up(run.idx, 1, kWave)};
    if (lane == 0) run = Pair{kNone, kNone};
    __syncthreads();
    for (uint32_t wv = 0; wv < wave; ++wv) run = pair_min(run, Pair{L.range[wv].lo, L.range[wv].hi});
    uint32_t on = 0;                                    // bit q: record q is on the front
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        on |= t * PER + q < cnt && !less_than(run, v[q]) ? 1u << q : 0u;
        run = pair_min(run, v[q]);
    }
    const uint32_t mine = (uint32_t)__popc(on), incl = wave_scan_sum(mine);
    if (lane == kWave - 1) L.tmp[wave] = incl;
    __syncthreads();
    uint32_t at = incl - mine, total = 0;
    for (uint32_t wv = 0; wv < NT / kWave; ++wv) {
        at += wv < wave ? L.tmp[wv] : 0u;
        total += L.tmp[wv];
    }
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q)
        if ((on >> q) & 1u) emit(at++, L.row[t * PER + q]);
    return uniform(total);
}

// Up to 1024 records eight lanes for each; more of them one lane each where their bins hold kSparse members or fewer on average
// over the records (sum of squared bin counts <= kSparse * cnt), and otherwise by sorting.  Selections of 2048 (4096) rows, all on
// the front, in us, pairwise with one lane / by sorting: 48 members a bin 42 / 50 (74 / 87), 64 members 56 / 53 (100 / 93),
// 96 members 71 / 50 (131 / 88), 1024 members 615 / 54 (1219 / 95).
constexpr uint32_t kSparse = 64;
template <typename Emit>
__device__ inline uint32_t staged_front(FinishLds &L, uint32_t cnt, Emit &&emit) {
    if (cnt <= 1024) return staged_front_by<8>(L, cnt, emit);           // block-uniform
    constexpr uint32_t P = kPerFinish;
    const uint32_t t = thread_here();
    uint32_t sq = 0;                                    // at most cnt * kStage < 2^32
#pragma unroll
    for (uint32_t q = 0; q < P; ++q) {
        const uint32_t b = q * kFinishThreads + t;
        const uint32_t n = L.off[padded<P>(b + 1)] - L.off[padded<P>(b)];
        sq += n * n;
    }
    sq = wave_sum(sq);
    __syncthreads();                                    // L.tmp may still be read by the scan before
    if (t % kWave == 0) L.tmp[t / kWave] = sq;
    __syncthreads();
    uint32_t total = 0;
    for (uint32_t wv = 0; wv < kFinishThreads / kWave; ++wv) total += L.tmp[wv];
    return total <= kSparse * cnt ? staged_front_by<1>(L, cnt, emit) : sorted_front(L, cnt, emit);
}

// The front among up to kStage records held by the threads of the finishing block (record q of thread t is
// there when bit q of live is set; its row is row_of(q)); the tables are in their neutral states and the
// block has met since.  end: no record is past that many (record q of thread t counts as number q * kFinishThreads + t); registers
// without any cost a branch.  Any binning will do that is fine where the records are.  Calls emit(position, row) for every front
// member, position = its rank by (x, y, row), and returns their number.
template <typename RowOf, typename Emit>
__device__ inline uint32_t finish_in_lds(FinishLds &L, const Binning &bin, const uint64_t (&rx)[kStage / kFinishThreads],
                                         const uint64_t (&ry)[kStage / kFinishThreads], RowOf &&row_of, uint32_t live,
                                         uint32_t end, Emit &&emit) {
    static_assert(kFinishThreads == 1024, "kPerFinish assumes 1024 threads");
    constexpr uint32_t P = kPerFinish, PER = kStage / kFinishThreads;
    auto there = [&](uint32_t q) { return q * kFinishThreads < end; };             // (uniform)
    // Survivors that are dominated for sure are dropped first: those with a survivor of a strictly lower bin at or below their y,
    // and those that their own bin's representative dominates -- the survivor with the bin's least y (of those,
    // the least x); rows often tie in x, and then the representative settles all of them but the ties in y.
    // Tables: least y per bin in the LDS that the records are staged in afterwards, then its exclusive
    // prefix-min; the representatives' x in the LDS of the bin counts.
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q)
        if (there(q) && ((live >> q) & 1u)) atomicMin((unsigned long long *)&L.lower[padded<P>(bin(rx[q]))], (unsigned long long)ry[q]);
    __syncthreads();
    uint32_t least = 0;                                 // bit q: the record has its own bin's least y
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        if (!there(q)) break;
        const uint32_t b = bin(rx[q]);
        const bool is = ((live >> q) & 1u) && ry[q] == L.lower[padded<P>(b)];
        if (is) atomicMin((unsigned long long *)&L.rep[b], (unsigned long long)rx[q]);
        least |= is ? 1u << q : 0u;
    }
    __syncthreads();
    scan_min_excl<kFinishThreads>(L.lower, L.tmp64);
    uint32_t alive = 0;
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        if (!there(q)) break;
        const uint32_t b = bin(rx[q]);
        const uint64_t rep_x = L.rep[b];
        const bool by_rep = rep_x <= rx[q] && (rep_x < rx[q] || !((least >> q) & 1u));
        const bool is = ((live >> q) & 1u) && ry[q] < L.lower[padded<P>(b)] && !by_rep;
        if (is) atomicAdd(&L.off[padded<P>(b)], 1u);
        alive |= is ? 1u << q : 0u;
    }
    __syncthreads();                                    // both tables have been read by everyone: records may be staged from here on
    scan_sum_excl<kFinishThreads, true>(L.off, L.tmp);
    const uint32_t m_alive = uniform(L.off[padded<P>(kBins)]);
    // records staged in LDS, grouped by bin
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        if (there(q) && ((alive >> q) & 1u)) {
            const uint32_t b = bin(rx[q]), pos = L.off[padded<P>(b)] + atomicAdd(&L.cur[b], 1u);
            L.kx[pos] = rx[q]; L.ky[pos] = ry[q]; L.row[pos] = row_of(q); L.bin[pos] = (uint16_t)b;
        }
    }
    return staged_front(L, m_alive, emit);
}

__device__ inline void finish_tables_neutral(FinishLds &L) {
    constexpr uint32_t P = kPerFinish;
    const uint32_t t = thread_here();
    for (uint32_t i = t; i < padded_size<P>(); i += kFinishThreads) L.lower[i] = kNone;
#pragma unroll
    for (uint32_t q = 0; q < kPerFinish; ++q) {
        const uint32_t i = q * kFinishThreads + t;
        L.rep[i] = kNone;
        L.cur[i] = 0;
        L.off[padded<P>(i)] = 0;
        L.foff[padded<P>(i)] = 0;
    }
    if (t == 0) L.nfront = 0;
}

// More kept rows than one block takes alone are finished by the n_parts blocks of the launch (part =
// 0 .. n_parts - 1).  Bins are independent until positions in the output are handed out, so each part takes a
// run of consecutive bins that holds about m / n_parts kept rows (bin b belongs to part floor(first kept-row
// slot of b * n_parts / m)), drops what a kept row of a lower bin dominates (large_survivors), finds the front members among
// the rest, and writes their rows, in order, to the workspace from its first slot on.  No part waits for
// another: each ends by taking a ticket, and the part that draws the last one lines the parts' runs up in
// the output (large_gather).
// Bound by latency: two passes over the kept rows' keys and a dozen steps between barriers.  8 500 kept rows, front of 2 820:
// 28 us; 74 us with three passes, dominated records staged as well and the parts' runs copied one after the other.
constexpr uint32_t kLargeParts = 64;                    // blocks that finish a large front (the finishing block is one)
constexpr uint32_t kLargeBatch = 10;                    // records per thread requested at a time
static_assert(kLargeParts <= kWave, "the last part scans the parts' counts in one wave");
static_assert(kLargeParts <= sizeof(SelectScratch::part_cnt) / sizeof(uint32_t), "one scratch entry per part");
struct LargePart {
    Stretch of;                 // what its bins slice
    uint32_t g_lo;              // its first slot
    uint32_t n_alive;           // its survivors: their positions are at w.staged[g_lo ..]
};
// The tables must be in their neutral states, and the block has met since.
__device__ inline LargePart large_survivors(FinishLds &L, const ParetoWs &w, const Binning &bin, uint32_t m, uint32_t part,
                                            uint32_t n_parts) {
    constexpr uint32_t P = kPerFinish, NT = kFinishThreads, B = kLargeBatch;
    const uint32_t t = threadIdx.x, lane = t % kWave;
    const bool held = m <= B * NT;                      // one batch: the second pass finds the keys in registers
    if (t == 0) {
        L.first = kBins;
        L.last = 0;
        L.alive = 0;
    }
    // The end of a batch can be beyond 32 bits; sums that saturate are past every row then (there are at most 2^32 - 4096).
    auto plus = [](uint32_t q, uint32_t d) { return __builtin_elementwise_add_sat(q, d); };
    uint64_t kx[B], ky[B];
    auto request = [&](uint32_t q0) {
#pragma unroll
        for (uint32_t u = 0; u < B; ++u) {
            const uint32_t q = plus(q0, u * NT) < m ? q0 + u * NT : 0u;
            kx[u] = w.skx[q];
            ky[u] = w.sky[q];
        }
    };
    request(t);
    __syncthreads();
    // One pass over all kept rows: rows per bin and the least y per bin, both in LDS (the latter where
    // records are staged afterwards).
    for (uint32_t q0 = t; q0 < m;) {
#pragma unroll
        for (uint32_t u = 0; u < B; ++u) {
            if (plus(q0, u * NT) < m) {
                const uint32_t b = padded<P>(bin(kx[u]));
                atomicAdd(&L.off[b], 1u);
                atomicMin((unsigned long long *)&L.lower[b], (unsigned long long)ky[u]);
            }
        }
        q0 = plus(q0, B * NT);
        if (q0 < m) request(q0);
    }
    __syncthreads();
    scan_sum_excl<NT, true>(L.off, L.tmp);              // entry kBins = m
    scan_min_excl<NT>(L.lower, L.tmp64);                // least y among the kept rows of strictly lower bins
#pragma unroll
    for (uint32_t q = 0; q < P; ++q) {
        const uint32_t i = q * NT + t, off = L.off[padded<P>(i)];
        if (L.off[padded<P>(i + 1)] != off && (uint32_t)((uint64_t)off * n_parts / m) == part) {
            atomicMin(&L.first, i);
            atomicMax(&L.last, i);
        }
    }
    __syncthreads();
    const uint32_t b_lo = uniform(L.first), b_hi = uniform(L.last);        // the part's bins (non-empty ones in between are all its own)
    LargePart r{stretch_of(bin, uniform(L.rng[1]), b_lo, b_hi), 0, 0};
    if (b_lo > b_hi) return r;                          // block-uniform
    r.g_lo = uniform(L.off[padded<P>(b_lo)]);
    // The part's kept rows that no kept row of a lower bin dominates: listed in the workspace.
    auto own = [&](uint32_t b) { return b >= b_lo && b <= b_hi; };
    for (uint32_t q0 = t; q0 < (m + NT - 1) / NT * NT; q0 = plus(q0, B * NT)) {      // wave-uniform trip count for the ballots
        if (!held) {                                    // block-uniform
#pragma unroll
            for (uint32_t u = 0; u < B; ++u) kx[u] = w.skx[plus(q0, u * NT) < m ? q0 + u * NT : 0u];
#pragma unroll
            for (uint32_t u = 0; u < B; ++u)
                if (plus(q0, u * NT) < m && own(bin(kx[u]))) ky[u] = w.sky[q0 + u * NT];
        }
#pragma unroll
        for (uint32_t u = 0; u < B; ++u) {
            const uint32_t b = bin(kx[u]);
            const bool alive = plus(q0, u * NT) < m && own(b) && ky[u] < L.lower[padded<P>(b)];
            const uint64_t mask = __ballot(alive);
            if (mask == 0) continue;                    // wave-uniform
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&L.alive, (uint32_t)__popcll(mask));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(mask & ((1ull << lane) - 1));
            if (alive) w.staged[r.g_lo + at] = q0 + u * NT;
        }
    }
    __syncthreads();
    r.n_alive = uniform(L.alive);
    return r;
}

// The range of the records of all threads, in every thread.  Contains a block barrier.
__device__ inline KeyRange block_range(FinishLds &L, KeyRange r) {
    constexpr uint32_t nw = kFinishThreads / kWave;
    const uint32_t t = thread_here();
    auto wave_range = [](const KeyRange &v) { return KeyRange{wave_min(v.lo), ~wave_min(~v.hi), wave_min(v.y)}; };
    r = wave_range(r);
    if (t % kWave == 0) L.range[t / kWave] = r;
    __syncthreads();
    return wave_range(L.range[t % nw]);
}
__device__ inline Binning binning_of(const KeyRange &r) { return r.lo <= r.hi ? binning_of(r.lo, r.hi) : binning_of(0, kNone); }
// Bins for a part's records: over their range inside the part's stretch of the common bins, when there are any.  A row far beyond
// the sampled range shares the first or the last of the common bins; over its range the part's others would share one bin.
__device__ inline Binning binning_of(const KeyRange &r, const Stretch &of) {
    const uint64_t lo = r.lo < of.lo ? of.lo : r.lo, hi = min_u64(r.hi, of.hi);
    return lo <= hi ? binning_of(lo, hi) : binning_of(r);
}

// The records of up to kStage survivors (row[q]: the position of record q, where bit q of live is set; 0 elsewhere), their rows
// in the place of the positions, and bins over their range inside `of`, or over all of it when more than a sixteenth of the n are
// outside (too many for the end bins).  Resets the tables, which the block has read; contains a block barrier.
__device__ inline Binning listed_records(FinishLds &L, const ParetoWs &w, uint64_t (&rx)[kStage / kFinishThreads],
                                         uint64_t (&ry)[kStage / kFinishThreads], uint32_t (&row)[kStage / kFinishThreads],
                                         uint32_t live, uint32_t n, const Stretch &of) {
    constexpr uint32_t PER = kStage / kFinishThreads;
    KeyRange r = KeyRange::none();
    uint32_t outside = 0;                               // records of the wave
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        rx[q] = w.skx[row[q]];
        ry[q] = w.sky[row[q]];
        row[q] = w.surv[row[q]];
    }
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const bool there = (live >> q) & 1u;
        if (there) r.add(rx[q], kNone);
        outside += (uint32_t)__popcll(__ballot(there && (rx[q] < of.lo || rx[q] > of.hi)));
    }
    finish_tables_neutral(L);
    const uint32_t t = thread_here();
    if (t % kWave == 0) L.tmp64[t / kWave] = outside;    // (L.tmp may still be read by a round's start)
    r = block_range(L, r);
    outside = wave_sum(t % kWave < kFinishThreads / kWave ? (uint32_t)L.tmp64[t % kWave] : 0u);
    return 16 * outside <= n ? binning_of(r, of) : binning_of(r);
}

// A part with more survivors than the staging arrays hold (their positions listed in w.staged[g_lo ..]): prunes and
// groups them by x, so that they can be finished in rounds of consecutive groups.  Leaves their positions in w.grouped[g_lo ..],
// a slot each (kNoSurvivor: none, or one that was pruned), and marks in w.staged[g_lo ..] where a group begins (no mark: 0); every group
// has fewer than kStage slots.  Returns the number of slots.
// The survivors are pruned and grouped by 4096 bins over their range inside the part's stretch; a bin that holds kStage or
// more is done likewise, with bins over its range, and so on: ranges are 2^12 times smaller each time (after the first), so
// seven times are the most until a bin is one x.  Then only those with the least y are left, which are equal, and grouped by row.
// Bins that wait for this are a list, its links in the first two entries of the bins' stretches of w.staged.  (There are at most
// 2^32 - 4096 rows: indices below do not wrap.)
// (1.9 million front rows: 2.6 ms; 40 ms with the bins that all parts share, which hold front / 4096 rows and more each.  One row far
// from all others collapses the first bins: 600 000 front rows 0.90 ms without one, 0.90 - 0.93 ms with one, and 4.4 - 37 ms when a
// bin beyond LDS is tested pair by pair, which takes minutes for some hundred thousand rows of the same x.)
constexpr uint32_t kNoSurvivor = ~0u;
__device__ inline uint32_t large_group(FinishLds &L, const ParetoWs &w, const LargePart &part) {
    constexpr uint32_t P = kPerFinish, NT = kFinishThreads, B = 4;
    const uint32_t t = threadIdx.x;
    uint32_t *list = w.staged + part.g_lo, *grouped = w.grouped + part.g_lo;
    uint32_t slots = 0;
    if (t == 0) L.todo = kNoSurvivor;
    uint32_t at = 0, cnt = part.n_alive;                // in work: list[at .. at + cnt)
    for (bool whole = true;; whole = false) {
        auto records = [&](auto &&use) {                // use(position, kx, ky) for each of them, B in flight
            for (uint32_t i0 = t; i0 < cnt; i0 += B * NT) {
                uint32_t q[B];
                uint64_t kx[B], ky[B];
#pragma unroll
                for (uint32_t u = 0; u < B; ++u) q[u] = list[at + (i0 + u * NT < cnt ? i0 + u * NT : i0)];
#pragma unroll
                for (uint32_t u = 0; u < B; ++u) {
                    kx[u] = w.skx[q[u]];
                    ky[u] = w.sky[q[u]];
                }
#pragma unroll
                for (uint32_t u = 0; u < B; ++u)
                    if (i0 + u * NT < cnt) use(q[u], kx[u], ky[u]);
            }
        };
        KeyRange r = KeyRange::none();
        records([&](uint32_t, uint64_t kx, uint64_t ky) { r.add(kx, ky); });
        finish_tables_neutral(L);                       // (the tables have been read by everybody)
        r = block_range(L, r);
        const bool one_x = r.lo == r.hi;                // block-uniform
        Binning bin = whole ? binning_of(r, part.of) : binning_of(r);
        if (one_x) {
            KeyRange rows = KeyRange::none();
            records([&](uint32_t q, uint64_t, uint64_t ky) {
                if (ky == r.y) rows.add(w.surv[q], 0);
            });
            __syncthreads();
            bin = binning_of(block_range(L, rows));
        } else {
            records([&](uint32_t, uint64_t kx, uint64_t ky) {
                atomicMin((unsigned long long *)&L.lower[padded<P>(bin(kx))], (unsigned long long)ky);
            });
            __syncthreads();
            scan_min_excl<NT>(L.lower, L.tmp64);
        }
        auto kept = [&](auto &&use) {                   // use(position, bin)
            records([&](uint32_t q, uint64_t kx, uint64_t ky) {
                if (one_x) {
                    if (ky == r.y) use(q, bin(w.surv[q]));
                } else {
                    const uint32_t b = bin(kx);
                    if (ky < L.lower[padded<P>(b)]) use(q, b);
                }
            });
        };
        kept([&](uint32_t, uint32_t b) { atomicAdd(&L.off[padded<P>(b)], 1u); });
        __syncthreads();
        scan_sum_excl<NT, true>(L.off, L.tmp);
        kept([&](uint32_t q, uint32_t b) { grouped[at + L.off[padded<P>(b)] + atomicAdd(&L.cur[b], 1u)] = q; });
        __syncthreads();                                // the list has been read
        const uint32_t left = uniform(L.off[padded<P>(kBins)]);
        if (whole) slots = cnt = left;
        for (uint32_t i = t; i < cnt; i += NT) {
            list[at + i] = i < left ? 0u : 1u;          // (what is not left may be split anywhere)
            if (i >= left) grouped[at + i] = kNoSurvivor;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < P; ++q) {
            const uint32_t b = q * NT + t, first = L.off[padded<P>(b)], members = L.off[padded<P>(b + 1)] - first;
            if (members >= kStage) {
                list[at + first + 1] = members;
                list[at + first] = atomicExch(&L.todo, at + first);
            } else if (members) {
                list[at + first] = 1;
            }
        }
        __syncthreads();
        at = uniform(L.todo);
        if (at == kNoSurvivor) return slots;            // block-uniform
        const uint32_t next = list[at];
        cnt = uniform(list[at + 1]);
        __syncthreads();                                // everybody has read the link
        if (t == 0) L.todo = next;
        for (uint32_t i = t; i < cnt; i += NT) list[at + i] = grouped[at + i];
        __syncthreads();
    }
}

// The part's front when its survivors do not fit the staging arrays: groups of consecutive x, as many at a time as do.  Returns
// the number of members, whose rows are at w.staged[g_lo ..] in order.
__device__ inline uint32_t large_rounds(FinishLds &L, const ParetoWs &w, const LargePart &part) {
    constexpr uint32_t NT = kFinishThreads, PER = kStage / NT;
    const uint32_t slots = large_group(L, w, part);
    const uint32_t *grouped = w.grouped + part.g_lo, *begins = w.staged + part.g_lo;
    uint32_t n_front = 0;
    for (uint32_t from = 0; from < slots;) {
        const uint32_t t = thread_here(), left = slots - from;
        uint32_t end = 0;                               // the last group that begins within kStage slots
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint32_t i = q * NT + t;
            if (i < left && begins[from + i]) end = i;
        }
        end = wave_max(end);
        if (t % kWave == 0) L.tmp[t / kWave] = end;
        __syncthreads();                                // (also: the round before is done with the tables)
        end = left <= kStage ? left : wave_max(L.tmp[t % (NT / kWave)]);
        uint64_t rx[PER], ry[PER];
        uint32_t rr[PER], live = 0;
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint32_t i = q * NT + t;
            rr[q] = i < end ? grouped[from + i] : kNoSurvivor;
            live |= rr[q] != kNoSurvivor ? 1u << q : 0u;
            rr[q] = rr[q] != kNoSurvivor ? rr[q] : 0u;
        }
        const Binning bin = listed_records(L, w, rx, ry, rr, live, end, Stretch{0, kNone});
        n_front += finish_in_lds(L, bin, rx, ry, [&](uint32_t q) { return rr[q]; }, live, end, [&](uint32_t pos, uint32_t row) {
            w.staged[part.g_lo + n_front + pos] = row;  // (over marks of slots that are done with)
        });
        from += end;
    }
    return n_front;
}

// Draws the part's ticket; the block with the last one copies all parts' runs to the output.
__device__ inline void large_gather(FinishLds &L, const ParetoWs &w, SelectScratch *sc, uint32_t part, uint32_t n_parts,
                                    uint32_t g_lo, uint32_t n_front, uint64_t *out_idx, uint64_t capacity,
                                    uint64_t *out_count) {
    constexpr uint32_t NT = kFinishThreads;
    const uint32_t t = threadIdx.x, lane = t % kWave;
    if (t == 0) {
        sc->part_lo[part] = g_lo;
        sc->part_cnt[part] = n_front;
    }
    // The ticket: everything this part wrote is visible to the part that draws the last one.  One thread
    // fences for the block, after every thread's stores have been acknowledged and the block has met (a
    // fence per wave costs a cache write-back each: 1 024 of them took most of the kernel's time).
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (t == 0) {
        __threadfence();
        const bool last = atomicAdd(&sc->counters[1], 1u) == n_parts - 1;
        if (last) __threadfence();
        L.is_last = last ? 1u : 0u;
    }
    __syncthreads();
    if (!L.is_last) return;
    if (t < kWave) {
        const uint32_t c = t < n_parts ? sc->part_cnt[t] : 0u;
        const uint32_t incl = wave_scan_sum(c);
        L.part_base[t] = incl - c;
        L.part_cnt[t] = c;
        L.part_lo[t] = t < n_parts ? sc->part_lo[t] : 0u;
        if (t == kWave - 1) {
            out_count[0] = incl;
            sc->counters[1] = 0;
        }
    }
    __syncthreads();
    // Every wave copies the runs of kPerWave parts side by side, eight loads in flight (one part after the other is a chain of 64
    // memory latencies: 36 of 62 us for a front of 2800 rows).
    constexpr uint32_t kPerWave = kLargeParts / (NT / kWave), kDeep = 8 / kPerWave;
    static_assert(kPerWave * (NT / kWave) == kLargeParts && kPerWave * kDeep == 8, "all parts, eight loads");
    uint32_t most = 0;
#pragma unroll
    for (uint32_t j = 0; j < kPerWave; ++j) {
        const uint32_t c = L.part_cnt[t / kWave * kPerWave + j];
        most = c > most ? c : most;
    }
    for (uint32_t i0 = lane; i0 < most; i0 += kDeep * kWave) {
        uint32_t v[kPerWave][kDeep];
#pragma unroll
        for (uint32_t j = 0; j < kPerWave; ++j) {
            const uint32_t p = t / kWave * kPerWave + j, c = L.part_cnt[p], lo = L.part_lo[p];
#pragma unroll
            for (uint32_t u = 0; u < kDeep; ++u) v[j][u] = c ? w.staged[lo + (i0 + u * kWave < c ? i0 + u * kWave : c - 1)] : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < kPerWave; ++j) {
            const uint32_t p = t / kWave * kPerWave + j, c = L.part_cnt[p];
            const uint64_t base = L.part_base[p];
#pragma unroll
            for (uint32_t u = 0; u < kDeep; ++u) {
                const uint32_t i = i0 + u * kWave;
                if (i < c && base + i < capacity) out_idx[base + i] = v[j][u];
            }
        }
    }
}

// Blocks of the launch: 0 finishes the front; 1 runs a waiting top-k merge (only launched with one); the
// others return at once unless more than kStage rows survived, and then share the large front with block 0.
__global__ __launch_bounds__(kFinishThreads) void pareto_finish_kernel(ParetoWs w, uint32_t n, SelectScratch *sc,
                                                                        uint64_t *out_idx,
                                                                        uint64_t capacity, uint64_t *out_count,
                                                                        MergeRider rider) {
    const uint32_t first_helper = rider.n_blocks ? 2 : 1;
    if (rider.n_blocks && blockIdx.x == 1) {
        if (rider.K == 1)
            topk_merge_body<1, kFinishThreads>(rider.w, rider.n_blocks, rider.k, rider.out_idx, rider.out_val, rider.out_cnt);
        else if (rider.K == 2)
            topk_merge_body<2, kFinishThreads>(rider.w, rider.n_blocks, rider.k, rider.out_idx, rider.out_val, rider.out_cnt);
        else if (rider.K == 3)
            topk_merge_body<3, kFinishThreads>(rider.w, rider.n_blocks, rider.k, rider.out_idx, rider.out_val, rider.out_cnt);
        else
            topk_merge_body<4, kFinishThreads>(rider.w, rider.n_blocks, rider.k, rider.out_idx, rider.out_val, rider.out_cnt);
        return;
    }
    __shared__ FinishLds L;
    const uint32_t t = threadIdx.x;
    const bool helper = blockIdx.x >= first_helper;     // block-uniform
    if (helper && sc->counters[0] <= kStage) return;
    // Everything the finishing block reads from global memory is requested at once, before the survivor
    // count is known: the first kStage survivor records (index clamped to the workspace's n rows; entries
    // at or beyond the count are ignored later), the count and the sample partials.
    constexpr uint32_t kPer = kStage / kFinishThreads;
    uint64_t rx[kPer], ry[kPer];
    uint32_t rr[kPer];
    if (!helper) {
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            const uint32_t j = q * kFinishThreads + t, jc = j < n ? j : n - 1;
            rx[q] = w.skx[jc];
            ry[q] = w.sky[jc];
            rr[q] = w.surv[jc];
        }
    }
    const uint32_t m = sc->counters[0];
    finish_tables_neutral(L);                           // while the loads are under way
    const Binning bin = sampled_binning(sc, L.rng);     // its barrier also covers the tables above
    const bool large = m > kStage;                      // block-uniform
    const uint32_t part = helper ? blockIdx.x - first_helper + 1 : 0, n_parts = gridDim.x - first_helper + 1;
    LargePart p{Stretch{0, kNone}, 0, m};
    if (large) p = large_survivors(L, w, bin, m, part, n_parts);
    uint32_t n_front;
    if (p.n_alive <= kStage) {                          // (a part without survivors goes through with no live record)
        uint32_t live = 0;
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) live |= q * kFinishThreads + t < p.n_alive ? 1u << q : 0u;
        Binning own = bin;
        if (large) {
            // Bins of the part's own: its share of the common ones is few, and one of those may hold hundreds of survivors (the
            // lowest ones, for want of lower bins that would prune them).
#pragma unroll
            for (uint32_t q = 0; q < kPer; ++q) rr[q] = (live >> q) & 1u ? w.staged[p.g_lo + q * kFinishThreads + t] : 0u;
            own = listed_records(L, w, rx, ry, rr, live, p.n_alive, p.of);
        }
        n_front = finish_in_lds(L, own, rx, ry, [&](uint32_t q) { return rr[q]; }, live, p.n_alive, [&](uint32_t pos, uint32_t row) {
            if (large) w.staged[p.g_lo + pos] = row;
            else if (pos < capacity) out_idx[pos] = row;
        });
    } else {
        n_front = large_rounds(L, w, p);
    }
    if (large) large_gather(L, w, sc, part, n_parts, p.g_lo, n_front, out_idx, capacity, out_count);
    else if (t == 0) out_count[0] = n_front;
}

// Selections over at most kStage rows: one launch without sample, filter pass and block partials.  Block 0 takes the
// Pareto selection (sel.pareto) with every passing row as a record; the next one (or block 0) the top-k of one group.
// Bound by latency.  1080 rows, both selections: 9.5 us, with the evaluation 13.4 us a call (12.6 and 15.7 us with the waves' totals gone
// through by every wave); filter pass and finishing kernel took 10.2 + 8.3 us, 25.4 us a call.  A front of 155 among 4096 rows alone: 15.7 us
// (17.6; 22.6 in three launches), so the line lies where the records stop fitting the finishing block.
struct SmallSelect {
    uint32_t pareto, k;                 // k = 0: no top-k
    const double *x, *y;
    RowFilter f;
    uint64_t *out_idx, capacity, *out_count;
    const double *obj;
    RowFilter top_f;
    uint64_t *top_idx;
    double *top_val;
    uint64_t *top_cnt;
};
template <int K>
__device__ inline void small_topk(const SmallSelect &s, uint32_t n) {
    constexpr int kNW = kFinishThreads / kWave;
    __shared__ Pair s_pairs[kNW][K];
    __shared__ uint32_t s_cnt[kNW];
    TopList<K> l;
    l.init();
    uint32_t cnt = 0;
    constexpr uint32_t kPer = kStage / kFinishThreads;
    Row r[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q)
        r[q] = load_row<false, GUIDE_MAX_CONSTRAINTS>(s.obj, nullptr, s.top_f, q * kFinishThreads + threadIdx.x, n);
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        if (r[q].pass) {
            ++cnt;
            l.insert_ascending(Pair{key_of(r[q].x), (uint64_t)(q * kFinishThreads + threadIdx.x)});
        }
    }
    const uint32_t wave_cnt = wave_sum(cnt);
    if (threadIdx.x % kWave == 0) s_cnt[threadIdx.x / kWave] = wave_cnt;
    block_topk<K, kNW>(l, s_pairs, [&](int j, const Pair &p) {
        if ((uint32_t)j < s.k) {
            s.top_idx[j] = p.idx;
            s.top_val[j] = p.idx == kNone ? INFINITY : value_of(p.key);
        }
    });                                                 // (contains the barrier that publishes s_cnt)
    if (threadIdx.x == 0) {
        uint64_t c = 0;
        for (int wv = 0; wv < kNW; ++wv) c += s_cnt[wv];
        s.top_cnt[0] = c;
    }
}
__global__ __launch_bounds__(kFinishThreads) void small_select_kernel(SmallSelect s, uint32_t n) {
    if (!s.pareto || blockIdx.x == 1) {                 // block-uniform
        if (s.k == 1) small_topk<1>(s, n);
        else if (s.k == 2) small_topk<2>(s, n);
        else if (s.k == 3) small_topk<3>(s, n);
        else small_topk<4>(s, n);
        return;
    }
    __shared__ FinishLds L;
    __shared__ Pair s_best[kFinishThreads / kWave];
    constexpr uint32_t kPer = kStage / kFinishThreads;
    const uint32_t t = threadIdx.x;
    Row r[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q)
        r[q] = load_row<true, GUIDE_MAX_CONSTRAINTS>(s.x, s.y, s.f, q * kFinishThreads + t, n);
    finish_tables_neutral(L);
    uint64_t rx[kPer], ry[kPer], lo = kNone;
    uint32_t live = 0;
    Pair best = {kNone, kNone};                         // (y key, x key) of the least y
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        rx[q] = ry[q] = 0;
        if (q * kFinishThreads >= n) continue;          // (uniform)
        const bool there = r[q].pass;
        live |= there ? 1u << q : 0u;
        rx[q] = there ? key_of(r[q].x) : 0;
        ry[q] = there ? key_of(r[q].y) : 0;
        lo = there ? min_u64(lo, rx[q]) : lo;
        if (there) best = pair_min(best, Pair{ry[q], rx[q]});
    }
    lo = wave_min(lo);
    best = wave_min(best);
    if (t % kWave == 0) {
        L.tmp64[t / kWave] = lo;
        s_best[t / kWave] = best;
    }
    __syncthreads();
    if (t < kWave) {
        constexpr uint32_t kNW = kFinishThreads / kWave;
        lo = wave_min(t < kNW ? L.tmp64[t] : kNone);
        best = wave_min(t < kNW ? s_best[t] : Pair{kNone, kNone});
        if (t == 0) {
            L.rng[0] = lo;
            L.rng[1] = best.idx;
        }
    }
    __syncthreads();
    lo = uniform(L.rng[0]);
    if (lo == kNone) {                                  // no row passes (uniform)
        if (t == 0) s.out_count[0] = 0;
        return;
    }
    const uint32_t n_front = finish_in_lds(L, binning_of(lo, uniform(L.rng[1])), rx, ry, [&](uint32_t q) { return q * kFinishThreads + t; },
                                           live, n, [&](uint32_t pos, uint32_t row) { if (pos < s.capacity) s.out_idx[pos] = row; });
    if (t == 0) s.out_count[0] = n_front;
}

__global__ void pareto_empty_kernel(uint64_t *out_count) { out_count[0] = 0; }

// A row chunk asked for by the caller is taken when batches of 8 or of 6 rows per thread tile it; otherwise the
// passes deal their own batches.  Calls fn(chunk, integral_constant<rows per thread>).
template <typename F>
void with_row_chunk(uint32_t row_chunk, F &&fn) {
    if (row_chunk && row_chunk % (kBlock * 8) == 0) fn(row_chunk, std::integral_constant<uint32_t, 8>{});
    else if (row_chunk && row_chunk % (kBlock * 6) == 0) fn(row_chunk, std::integral_constant<uint32_t, 6>{});
    else fn(kDefaultChunk, std::integral_constant<uint32_t, 8>{});
}

template <int K>
void launch_top1_pass(const guide_select_spec &spec, uint64_t n, void *ws, const SampleRider &sample, hipStream_t stream,
                      uint32_t row_chunk) {
    const uint32_t nb = blocks_for(n);
    with_max_constraints(spec.n_constraints, [&](auto maxc) {
        with_row_chunk(row_chunk, [&](uint32_t chunk, auto u) {
            hipLaunchKernelGGL((topk_pass_kernel<K, decltype(maxc)::value, decltype(u)::value>),
                               dim3(nb + (sample.on ? kSampleBlocks : 0)), dim3(kBlock), 0, stream, spec.objective,
                               make_filter(spec), (uint32_t)n, top1_ws(ws), nb, sample, chunk);
        });
    });
}
// Pairs per block partial for a request of k (the pass kernel's template argument).
int partial_width(uint32_t k) { return k <= 4 ? (int)k : 8; }
void launch_top1_pass(const guide_select_spec &spec, uint64_t n, void *ws, const SampleRider &sample, hipStream_t stream,
                      uint32_t chunk = 0) {
    switch (partial_width(spec.k)) {
        case 1: launch_top1_pass<1>(spec, n, ws, sample, stream, chunk); break;
        case 2: launch_top1_pass<2>(spec, n, ws, sample, stream, chunk); break;
        case 3: launch_top1_pass<3>(spec, n, ws, sample, stream, chunk); break;
        case 4: launch_top1_pass<4>(spec, n, ws, sample, stream, chunk); break;
        default: launch_top1_pass<8>(spec, n, ws, sample, stream, chunk); break;
    }
}
void launch_top1_merge(int K, void *ws, uint32_t n_blocks, uint32_t k, const guide_select_out &out, hipStream_t stream) {
    const Top1Ws w = top1_ws(ws);
    const dim3 one(1), nt(kMergeThreads);
    switch (K) {
        case 1: hipLaunchKernelGGL(topk_merge_kernel<1>, one, nt, 0, stream, w, n_blocks, k, out.idx, out.val, out.count); break;
        case 2: hipLaunchKernelGGL(topk_merge_kernel<2>, one, nt, 0, stream, w, n_blocks, k, out.idx, out.val, out.count); break;
        case 3: hipLaunchKernelGGL(topk_merge_kernel<3>, one, nt, 0, stream, w, n_blocks, k, out.idx, out.val, out.count); break;
        case 4: hipLaunchKernelGGL(topk_merge_kernel<4>, one, nt, 0, stream, w, n_blocks, k, out.idx, out.val, out.count); break;
        default: hipLaunchKernelGGL(topk_merge_kernel<8>, one, nt, 0, stream, w, n_blocks, k, out.idx, out.val, out.count); break;
    }
}

}  // namespace

static_assert(sizeof(SelectScratch) <= kSelectScratchMax, "kSelectScratchMax is too small");
size_t select_scratch_bytes() { return sizeof(SelectScratch); }


size_t select_workspace_bytes(const guide_select_spec &spec, uint64_t n) {
    if (spec.mode == GUIDE_SELECT_PARETO) return pareto_ws_bytes(n);
    const size_t a = topk_ws_bytes(spec.n_groups ? spec.n_groups : 1), b = top1_ws_bytes();
    return a > b ? a : b;
}

// Up to kStage rows (what the finishing block holds in LDS) and k <= 4 (wider lists of 16 waves do not fit the block
// merge): one launch.  1000 .. 4096 rows: a front 12.8 - 21.0 us against 20.5 - 30.1 us in three launches, a top-k 5.0 - 8.7
// against 6.5 - 11.5 us in two.
bool select_is_small(uint64_t n) { return n > 0 && n <= kStage; }
static hipError_t launch_small(const guide_select_spec *topk, const guide_select_out *topk_out, const guide_select_spec *pareto,
                               const guide_select_out *pareto_out, uint64_t n, hipStream_t stream) {
    SmallSelect s;
    memset(&s, 0, sizeof s);
    if (pareto) {
        s.pareto = 1;
        s.x = pareto->objective;
        s.y = pareto->objective_y;
        s.f = make_filter(*pareto);
        s.out_idx = pareto_out->idx;
        s.capacity = pareto_out->capacity;
        s.out_count = pareto_out->count;
    }
    if (topk) {
        s.k = topk->k;
        s.obj = topk->objective;
        s.top_f = make_filter(*topk);
        s.top_idx = topk_out->idx;
        s.top_val = topk_out->val;
        s.top_cnt = topk_out->count;
    }
    hipLaunchKernelGGL(small_select_kernel, dim3(pareto && topk ? 2 : 1), dim3(kFinishThreads), 0, stream, s, (uint32_t)n);
    return hipGetLastError();
}

hipError_t launch_select_topk(const guide_select_spec &spec, uint64_t n, const guide_select_out &out, void *ws,
                              void *scratch, hipStream_t stream) {
    (void)scratch;
    if (!spec.group && select_is_small(n) && spec.k <= 4) return launch_small(&spec, &out, nullptr, nullptr, n, stream);
    if (!spec.group) {
        launch_top1_pass(spec, n, ws, SampleRider{}, stream);
        launch_top1_merge(partial_width(spec.k), ws, blocks_for(n), spec.k, out, stream);
        return hipGetLastError();
    }
    const uint32_t G = spec.n_groups, k = spec.k, nb = k == 1 ? blocks_for(n) : group_blocks(n, k);
    const GroupWs w = group_ws(ws, G, k, nb);
    const size_t lds = kGroupLdsBytes * G;
    with_max_constraints(spec.n_constraints, [&](auto maxc) {
        if (k == 1)
            hipLaunchKernelGGL((topk_group_first_kernel<decltype(maxc)::value>), dim3(nb), dim3(kBlock), 0, stream, spec.objective,
                               make_filter(spec), spec.group, G, (uint32_t)n, w);
        else
            hipLaunchKernelGGL((topk_group_kernel<decltype(maxc)::value>), dim3(nb), dim3(kGroupThreads), lds, stream,
                               spec.objective, make_filter(spec), spec.group, G, k, (uint32_t)n, w);
    });
    const dim3 groups(G), block(kBlock);
    switch (partial_width(k)) {
        case 1: hipLaunchKernelGGL(topk_group_merge_kernel<1>, groups, block, 0, stream, w, nb, k, out.idx, out.val, out.count); break;
        case 2: hipLaunchKernelGGL(topk_group_merge_kernel<2>, groups, block, 0, stream, w, nb, k, out.idx, out.val, out.count); break;
        case 3: hipLaunchKernelGGL(topk_group_merge_kernel<3>, groups, block, 0, stream, w, nb, k, out.idx, out.val, out.count); break;
        case 4: hipLaunchKernelGGL(topk_group_merge_kernel<4>, groups, block, 0, stream, w, nb, k, out.idx, out.val, out.count); break;
        default: hipLaunchKernelGGL(topk_group_merge_kernel<8>, groups, block, 0, stream, w, nb, k, out.idx, out.val, out.count); break;
    }
    return hipGetLastError();
}

// A launch with the timing events attached to its dispatch when there are any.
template <typename Kernel, typename... Args>
static void launch_timed(Kernel kernel, dim3 grid, dim3 block, hipStream_t stream, const LaunchTiming *tm, Args... args) {
    if (tm && tm->start) hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, tm->start, tm->stop, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, 0, stream, args...);
}

// The passes after the row sample: the filter pass (with the per-lane lists of a top-k that shares the
// columns) and the finishing kernel.  tm: two event pairs (filter, finish) or none.
static hipError_t launch_pareto_passes(const guide_select_spec &spec, uint64_t n, const guide_select_out &out, void *ws,
                                       SelectScratch *sc, const MergeRider &rider, hipStream_t stream,
                                       const SharedTopk *shared = nullptr, int shared_k = 0, uint32_t row_chunk = 0,
                                       const LaunchTiming *tm = nullptr) {
    const LaunchTiming *tm_filter = tm, *tm_fin = tm ? tm + 1 : nullptr;
    const ParetoWs w = pareto_ws(ws, n);
    const RowFilter f = make_filter(spec);
    const uint32_t nb = pareto_blocks(n), n32 = (uint32_t)n;
    const double *x = spec.objective, *y = spec.objective_y;
    const dim3 grid(nb), block(kBlock);
    with_row_chunk(row_chunk, [&](uint32_t chunk, auto u) {
        constexpr uint32_t U = decltype(u)::value;
        if (shared) {       // only offered for a Pareto selection without constraint columns
            const SharedTopk t = *shared;
            if (shared_k == 1) launch_timed(pareto_filter_kernel<0, 1, U>, grid, block, stream, tm_filter, x, y, f, n32, w, sc, t, chunk);
            else if (shared_k == 2) launch_timed(pareto_filter_kernel<0, 2, U>, grid, block, stream, tm_filter, x, y, f, n32, w, sc, t, chunk);
            else if (shared_k == 3) launch_timed(pareto_filter_kernel<0, 3, U>, grid, block, stream, tm_filter, x, y, f, n32, w, sc, t, chunk);
            else launch_timed(pareto_filter_kernel<0, 4, U>, grid, block, stream, tm_filter, x, y, f, n32, w, sc, t, chunk);
            return;
        }
        with_max_constraints(f.n_con, [&](auto maxc) {
            constexpr uint32_t MAXC = decltype(maxc)::value;
            launch_timed(pareto_filter_kernel<MAXC, 0, U>, grid, block, stream, tm_filter, x, y, f, n32, w, sc, SharedTopk{},
                         chunk);
        });
    });
    const uint32_t helpers = n > kStage ? kLargeParts - 1 : 0;     // no more than kStage rows: the staged path for sure
    launch_timed(pareto_finish_kernel, dim3((rider.n_blocks ? 2 : 1) + helpers), dim3(kFinishThreads), stream, tm_fin, w, n32,
                 sc, out.idx, out.capacity, out.count, rider);
    return hipGetLastError();
}

hipError_t launch_select_pareto(const guide_select_spec &spec, uint64_t n, const guide_select_out &out, void *ws,
                                void *scratch, hipStream_t stream) {
    if (n == 0) {
        hipLaunchKernelGGL(pareto_empty_kernel, dim3(1), dim3(1), 0, stream, out.count);
        return hipGetLastError();
    }
    if (select_is_small(n)) return launch_small(nullptr, nullptr, &spec, &out, n, stream);
    SelectScratch *sc = (SelectScratch *)scratch;
    hipLaunchKernelGGL(pareto_prepare_kernel, dim3(kSampleBlocks), dim3(kBlock), 0, stream, spec.objective,
                       spec.objective_y, make_filter(spec), (uint32_t)n, sc);
    return launch_pareto_passes(spec, n, out, ws, sc, MergeRider{}, stream);
}

// True when the top-k selection reads only the Pareto selection's x, y and flag columns (and the Pareto
// selection has no constraint columns); fills the description for the filter pass.
static bool shares_columns(const guide_select_spec &topk, const guide_select_spec &pareto, SharedTopk *t) {
    const double *x = pareto.objective, *y = pareto.objective_y;
    if (pareto.n_constraints != 0 || topk.n_constraints > 2 || topk.k > 4) return false;
    if (topk.objective != x && topk.objective != y) return false;
    if (topk.feasible && topk.feasible != pareto.feasible) return false;
    memset(t, 0, sizeof *t);
    t->obj_is_y = topk.objective == y ? 1u : 0u;
    t->use_feasible = topk.feasible ? 1u : 0u;
    t->n_con = topk.n_constraints;
    for (uint32_t c = 0; c < topk.n_constraints; ++c) {
        const double *col = topk.constraints[c].column;
        if (col != x && col != y) return false;
        t->con_is_y[c] = col == y ? 1u : 0u;
        t->cap[c] = topk.constraints[c].cap;
    }
    return true;
}

// A top-k selection (one group) and a Pareto selection over the same n > 0 rows in three launches
// instead of five.  The top-k merge rides along with the finishing kernel of the Pareto front (for block
// partials of up to 4 pairs; wider ones merge alone).  When the top-k reads only the Pareto selection's
// columns, its pass is folded into the filter pass (sample, filter + lists, finish + merge); otherwise the
// Pareto row sample rides along with the top-k pass (pass + sample, filter, finish + merge).
// sampled: the caller's own kernel has taken the row sample.
hipError_t launch_select_both(const guide_select_spec &topk, const guide_select_out &topk_out, void *topk_ws,
                              const guide_select_spec &pareto, const guide_select_out &pareto_out, void *pareto_ws_,
                              uint64_t n, void *scratch, hipStream_t stream, bool sampled,
                              uint32_t row_chunk, const LaunchTiming *pass_timing) {
    if (select_is_small(n) && topk.k <= 4) return launch_small(&topk, &topk_out, &pareto, &pareto_out, n, stream);
    SelectScratch *sc = (SelectScratch *)scratch;
    const int K = partial_width(topk.k);
    SharedTopk shared;
    const bool folded = shares_columns(topk, pareto, &shared);
    if (folded) {
        shared.w = top1_ws(topk_ws);
        if (!sampled)
            hipLaunchKernelGGL(pareto_prepare_kernel, dim3(kSampleBlocks), dim3(kBlock), 0, stream, pareto.objective,
                               pareto.objective_y, make_filter(pareto), (uint32_t)n, sc);
    } else {
        const SampleRider sample{sampled ? 0u : 1u, pareto.objective, pareto.objective_y, make_filter(pareto), sc};
        launch_top1_pass(topk, n, topk_ws, sample, stream, row_chunk);
    }
    MergeRider rider{};
    if (K <= 4)
        rider = MergeRider{top1_ws(topk_ws), folded ? pareto_blocks(n) : blocks_for(n), topk.k, (uint32_t)K, topk_out.idx,
                           topk_out.val, topk_out.count};       // partials: one per block of the kernel that kept the lists
    else
        launch_top1_merge(K, topk_ws, blocks_for(n), topk.k, topk_out, stream);
    return launch_pareto_passes(pareto, n, pareto_out, pareto_ws_, sc, rider, stream, folded ? &shared : nullptr, K, row_chunk,
                                pass_timing);
}

// The passes after the sample, for a caller whose own kernel has taken the row sample.
// merge_ws != nullptr: the merge of a folded top-k (merge_blocks block partials of kFusedTopK pairs) rides
// along with the finishing kernel instead of taking a launch of its own.
hipError_t launch_pareto_sampled(const guide_select_spec &spec, uint64_t n, const guide_select_out &out, void *ws,
                                 void *scratch, void *merge_ws, uint32_t merge_blocks,
                                 uint32_t merge_k, const guide_select_out *merge_out, hipStream_t stream,
                                 uint32_t row_chunk) {
    MergeRider rider{};
    if (merge_ws)
        rider = MergeRider{top1_ws(merge_ws), merge_blocks, merge_k, (uint32_t)kFusedTopK, merge_out->idx, merge_out->val,
                           merge_out->count};
    return launch_pareto_passes(spec, n, out, ws, (SelectScratch *)scratch, rider, stream, nullptr, 0, row_chunk);
}

size_t topk_partials_bytes() { return top1_ws_bytes(); }

// Merge of n_blocks block partials of kFusedTopK pairs each.
hipError_t launch_topk_merge(void *ws, uint32_t n_blocks, uint32_t k, const guide_select_out &out, hipStream_t stream) {
    launch_top1_merge(kFusedTopK, ws, n_blocks, k, out, stream);
    return hipGetLastError();
}

}  // namespace guide
