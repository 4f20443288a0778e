// IC kernels of the drawn-coins ("live") form: every arc's coin of a range of
// trials is drawn once, densely, into one bit row per trial, and a trial's
// cascade is then plain reachability over its live arcs, walked by one small
// workgroup per (trial, seed set) with the visited nodes as a bitmap in LDS.
//
// Coins depend on (rng_seed, trial, arc) only, so all seed sets of a call
// (common random numbers) share the rows: where a task that draws its own
// coins pays one hash block per (set, arc, 8 trials) examined, here a call
// pays one per (arc, 8 trials) whatever the number of sets, and an examined
// arc costs one bit.
#pragma once

#include "sim_kernels.hpp"

namespace imsim {

constexpr uint32_t kLiveQueues = 8;   // work queues, one per XCD (workgroup b runs on XCD b % 8)
constexpr uint32_t kCtlStep = 32;     // queue counters stand in 128-byte lines of their own
constexpr uint32_t kTinyCap = 16;     // nodes a lane follows alone before the cascade goes to a wavefront
constexpr uint32_t kTinySeeds = 4;    // larger seed sets go to a wavefront at once
constexpr uint32_t kTinyDeg = 256;    // coin-row form: so do nodes with more out-arcs
constexpr uint32_t kLaneArcs = 32;    // nodes with more live arcs are walked by their whole wavefront
constexpr uint32_t kLiveQ = 128;      // frontier entries of one level kept in LDS (the rest are read back from the list)
constexpr uint32_t kLiveBuf = 256;    // live arcs gathered per round and wavefront

constexpr uint32_t kHasArcs = 1u << 31;

// An arc's target with that node's own out-arcs: node (20 bits), first arc (24
// bits), out-degree (20 bits).  A cascade that meets the target has its row
// bounds at hand, one dependent read a step fewer than looking them up.
constexpr uint32_t kRecNodeBits = 20, kRecArcBits = 24;
__device__ __forceinline__ uint64_t arc_record(uint32_t v, uint32_t o0, uint32_t o1)
{
    return (uint64_t)v | ((uint64_t)o0 << kRecNodeBits) | ((uint64_t)(o1 - o0) << (kRecNodeBits + kRecArcBits));
}
__device__ __forceinline__ uint32_t rec_node(uint64_t r) { return (uint32_t)r & ((1u << kRecNodeBits) - 1u); }
__device__ __forceinline__ uint32_t rec_first(uint64_t r) { return (uint32_t)(r >> kRecNodeBits) & ((1u << kRecArcBits) - 1u); }
__device__ __forceinline__ uint32_t rec_degree(uint64_t r) { return (uint32_t)(r >> (kRecNodeBits + kRecArcBits)); }

__global__ __launch_bounds__(kBlock) void arc_record_kernel(const uint32_t* __restrict__ off, const uint32_t* __restrict__ idx, uint64_t m,
                                                            uint64_t* __restrict__ rec)
{
    for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < m; e += (uint64_t)gridDim.x * kBlock) {
        const uint32_t v = idx[e];
        rec[e] = arc_record(v, off[v], off[v + 1]);
    }
}

struct LiveParams {
    uint64_t n;
    const uint32_t* __restrict__ off;  // [n + 1] out-CSR offsets
    const uint32_t* __restrict__ idx;
    const uint64_t* __restrict__ rec;  // [m] arc records
    uint64_t m;
    uint64_t* rows;                    // [tc][row_words] coin bits of trial t0 + row, arc order
    uint64_t row_words;                // a multiple of 8
    uint32_t* rank;                    // [tc][row_words] live arcs before each coin word
    // the live graph of each trial: targets of its live arcs in arc order
    // (list_cap per trial) and, per node, where its own begin ([n + 1], with
    // kHasArcs when the node has out-arcs at all)
    uint32_t* loff;
    uint32_t* llist;
    uint64_t list_cap;
    uint32_t t0, tc;                   // trials of this range
    uint32_t T;
    // seed sets: set i's nodes are set_nodes[set_off[i] .. set_off[i + 1])
    const uint32_t* __restrict__ set_off;
    const uint32_t* __restrict__ set_nodes;
    uint32_t n_sets;
    const uint32_t* __restrict__ base;  // [tc][bitmap words] nodes active beforehand, or null
    uint32_t* todo;       // [tc][n_sets] sets whose cascade needs a workgroup
    uint32_t* todo_count; // [tc]
    uint32_t* taken;      // queue q (the rows q, q + kLiveQueues, ...): entries taken at kCtlStep * q
    uint32_t* entries;    // and entries listed at kCtlStep * q
    uint32_t take;        // entries taken at a time
    uint32_t* queue;      // [workgroup][n] nodes reached, in the order reached
    uint64_t* totals;          // [n_sets]
    uint32_t* set_node_counts; // [n_sets][n] or null
    uint32_t* status;
};

// Inclusive prefix sum over the wavefront's 64 lanes by DPP row shifts and
// row broadcasts (no LDS round trips, unlike ds_bpermute shuffles).
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x)
{
    int v = (int)x;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return (uint32_t)v;
}

// Wait for the wavefront's outstanding loads here.  Without it the compiler,
// which cannot see that a load behind a skipped branch has been waited for,
// waits for every store in turn in the branches that follow.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The rounds of philox4x64-10 that do not depend on the trial group: with
// counter (id, group, 0, 0) the first round's product of id, the second
// round's of what follows from it and the third round's first product are the
// same for every group, so an arc's eight blocks of a word share them.
struct PhiloxArc {
    uint64_t lo_a1;         // round 1: low product of id
    uint64_t hi_a1k;        // round 1: high product of id, ^ k1 (counter word 2 of round 2)
    uint64_t x0_3, x1_3;    // counter words 0, 1 of round 3 (before its key)
    uint64_t lo_a3, hi_a3;  // round 3: product of counter word 0
};

__device__ __forceinline__ PhiloxArc philox_arc(uint64_t id, uint64_t k0, uint64_t k1)
{
    PhiloxArc a;
    uint64_t hi;
    mul_wide_chain(id, kPhiloxM0, a.lo_a1, hi);
    a.hi_a1k = hi ^ k1;
    uint64_t lo_b, hi_b;
    mul_wide_chain(a.hi_a1k, kPhiloxM1, lo_b, hi_b);
    a.x0_3 = hi_b ^ (k0 + kWeyl0);
    a.x1_3 = lo_b;
    mul_wide_chain(a.x0_3, kPhiloxM0, a.lo_a3, a.hi_a3);
    return a;
}

__device__ __forceinline__ Block4 philox_group(const PhiloxArc& a, uint64_t group, uint64_t k0, uint64_t k1)
{
    // round 2's product of counter word 0 = group ^ k0 is uniform over the wavefront
    uint64_t lo_a2, hi_a2;
    mul_wide(kPhiloxM0, group ^ k0, lo_a2, hi_a2);
    k0 += 2 * kWeyl0;
    k1 += kWeyl1;
    uint64_t x2 = xor3_64(a.lo_a1, hi_a2, k1);
    k1 += kWeyl1;
    uint64_t lo_b, hi_b;
    mul_wide_chain(x2, kPhiloxM1, lo_b, hi_b);
    uint64_t x0 = xor3_64(hi_b, a.x1_3, k0);
    uint64_t x1 = lo_b;
    x2 = xor3_64(a.hi_a3, lo_a2, k1);
    uint64_t x3 = a.lo_a3;
#pragma unroll
    for (int r = 3; r < 10; ++r) {
        k0 += kWeyl0;
        k1 += kWeyl1;
        uint64_t lo_a, hi_a;
        mul_wide_chain(x0, kPhiloxM0, lo_a, hi_a);
        mul_wide_chain(x2, kPhiloxM1, lo_b, hi_b);
        x0 = xor3_64(hi_b, x1, k0);
        x2 = xor3_64(hi_a, x3, k1);
        x1 = lo_b;
        x3 = lo_a;
    }
    return Block4{x0, x1, x2, x3};
}

// Coin rows: a wavefront takes kChunks consecutive 64-arc chunks (lane = arc)
// and one 64-trial word.  A coin's compare over the wavefront is the
// 64-arc piece of that trial's row as it stands (no transpose); lane t keeps
// trial t's pieces and stores them together, eight of them as one 64-byte
// line.  Bound by the hash arithmetic (about 150 blocks a nanosecond) while
// there are wavefronts for the chip; few arcs take one chunk each (10,000
// arcs, 1,000 trials: 43 us with eight, 16 with one).
// `C` names outputs to zero here for the kernels that follow (total null: none).
struct LiveClear {
    uint32_t* status;       // four words, or null
    uint64_t* total;        // one
    uint32_t* node_counts;  // [n] or null
    uint64_t n;
};
template <uint32_t kChunks>
__global__ __launch_bounds__(kBlock) void live_draw_kernel(LiveClear C, uint64_t* __restrict__ rows, uint64_t row_words, const uint32_t* __restrict__ thr,
                                                           uint64_t m, uint32_t t0, uint32_t tc, uint64_t seed)
{
    const uint32_t lane = threadIdx.x & 63u;
    if (C.total) {
        if (C.status && blockIdx.x == 0 && threadIdx.x < 4) C.status[threadIdx.x] = 0;
        if (blockIdx.x == 0 && threadIdx.x == 4) *C.total = 0;
        if (C.node_counts)
            for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v < C.n; v += (uint64_t)gridDim.x * kBlock) C.node_counts[v] = 0;
    }
    const uint64_t wave = uniform64(((uint64_t)blockIdx.x * kBlock + threadIdx.x) >> 6);
    const uint64_t blocks8 = row_words / kChunks;
    const uint64_t words = (tc + 63) / 64;
    if (wave >= blocks8 * words) return;
    const uint64_t w = wave / blocks8, c8 = wave - w * blocks8;
    const uint32_t left = tc - (uint32_t)(64 * w);
    const uint32_t groups = left >= 64 ? 8u : (left + 7) / 8;
    const uint64_t g0 = t0 / 8 + 8 * w;  // t0 is a multiple of 64
    uint32_t lo[kChunks], hi[kChunks];
#pragma unroll
    for (uint32_t k = 0; k < kChunks; ++k) {
        lo[k] = 0;
        hi[k] = 0;
        const uint64_t e = (kChunks * c8 + k) * 64 + lane;
        const uint32_t th = e < m ? thr[e] : 0u;
        const uint64_t sure = __ballot(th == 0xFFFFFFFFu);
        if (__ballot(th != 0) == 0) continue;
        const PhiloxArc a = philox_arc(e, seed, kDomainIcArc);
        for (uint32_t g = 0; g < groups; ++g) {
            const Block4 b = philox_group(a, g0 + g, seed, kDomainIcArc);
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j) {
                const uint64_t row = __ballot(block_lane(b, j) < th) | sure;
                const bool mine = lane == 8 * g + j;
                lo[k] = mine ? (uint32_t)row : lo[k];
                hi[k] = mine ? (uint32_t)(row >> 32) : hi[k];
            }
        }
    }
    if (lane < left) {
        uint2* out = reinterpret_cast<uint2*>(rows + (64 * w + lane) * row_words + kChunks * c8);
        if constexpr (kChunks == 1) {
            out[0] = make_uint2(lo[0], hi[0]);
        } else {
#pragma unroll
            for (uint32_t k = 0; k < kChunks; k += 2)
                *reinterpret_cast<uint4*>(out + k) = make_uint4(lo[k], hi[k], lo[k + 1], hi[k + 1]);
        }
    }
}

// Per-trial bitmaps of a word-major state: out[row][v / 32] bit v % 32 = bit
// of trial t0 + row in A[w * n + v].  A wavefront transposes 64 nodes x 64 trials.
__global__ __launch_bounds__(kBlock) void live_base_kernel(const uint64_t* __restrict__ A, uint64_t n, uint32_t t0, uint32_t tc,
                                                           uint32_t* __restrict__ out, uint64_t bm_words)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t wave = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const uint64_t tiles = (n + 63) / 64;
    const uint64_t words = (tc + 63) / 64;
    if (wave >= tiles * words) return;
    const uint64_t w = wave / tiles, tile = wave - w * tiles;
    const uint64_t v = tile * 64 + lane;
    const uint64_t x = wave_transpose64(v < n ? A[(t0 / 64 + w) * n + v] : 0ull, lane);
    const uint64_t row = 64 * w + lane;
    if (row < tc) {
        out[row * bm_words + 2 * tile] = (uint32_t)x;
        out[row * bm_words + 2 * tile + 1] = (uint32_t)(x >> 32);
    }
}

// Live graphs: one workgroup per trial turns the coin row into a CSR of the
// live arcs alone.  A wavefront takes 64 coin words (lane = word), lays their
// set bits out densely in LDS (a prefix sum of the bit counts) and copies
// those arcs' targets; then every node's first live arc is the rank of its
// first coin bit.  A cascade reads two dependent words per node and live arc
// (bounds, target) from about 8 bytes per node of its trial, which stays in
// L2, where walking coin bits against the graph's own targets read three and
// missed L2 on every third access (200k nodes, 2M arcs, 128 sets x 1,000
// trials: 17.5 ms bound by 5.1 TB/s of such misses).
constexpr int kPackBlock = 512;
constexpr int kPackWaves = kPackBlock / 64;
__global__ __launch_bounds__(kPackBlock) void live_pack_kernel(LiveParams L)
{
    __shared__ uint32_t bufs[kPackWaves][kLiveBuf];
    __shared__ uint32_t sums[2][kPackWaves];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint64_t row = blockIdx.x;
    const uint64_t* bits = L.rows + row * L.row_words;
    uint32_t* rank = L.rank + row * L.row_words;
    uint32_t* loff = L.loff + row * (L.n + 1);
    uint32_t* llist = L.llist + row * L.list_cap;
    uint32_t* buf = bufs[wave];
    uint32_t before = 0;  // live arcs of the tiles behind
    uint32_t par = 0;
    uint64_t next = threadIdx.x < L.row_words ? bits[threadIdx.x] : 0ull;
    for (uint64_t x0 = 0; x0 < L.row_words; x0 += kPackBlock, par ^= 1u) {
        const uint64_t x = x0 + threadIdx.x;
        const uint64_t word = next;
        next = x + kPackBlock < L.row_words ? bits[x + kPackBlock] : 0ull;
        const uint32_t c = (uint32_t)__popcll(word);
        const uint32_t incl = wave_scan_incl(c);
        const uint32_t total = uniform32((uint32_t)__builtin_amdgcn_readlane((int)incl, 63));
        if (lane == 0) sums[par][wave] = total;
        __syncthreads();
        uint32_t at = before;
#pragma unroll
        for (uint32_t q = 0; q < kPackWaves; ++q) {
            const uint32_t y = sums[par][q];
            at += q < wave ? y : 0u;
            before += y;
        }
        at = uniform32(at);
        if (x < L.row_words) rank[x] = at + incl - c;
        for (uint32_t win = 0; win < total; win += kLiveBuf) {
            uint32_t p = incl - c - win;  // wraps below the window
            __builtin_amdgcn_wave_barrier();
            for (uint64_t b = word; b; b &= b - 1, ++p)
                if (p < kLiveBuf) buf[p] = (uint32_t)(64 * x) + (uint32_t)__builtin_ctzll(b);
            __builtin_amdgcn_wave_barrier();
            const uint32_t nn = total - win < kLiveBuf ? total - win : kLiveBuf;
#pragma unroll
            for (uint32_t y = 0; y < kLiveBuf / 64; ++y) {
                const uint32_t i = 64 * y + lane;
                if (i < nn && at + win + i < L.list_cap) llist[at + win + i] = L.idx[buf[i]];
            }
        }
    }
    __syncthreads();
    // (list_cap holds any count the coins bring about short of a 16-sigma
    // excess, which is reported like a cut-off run)
    if (before > L.list_cap) {
        if (threadIdx.x == 0) L.status[1] = 1;
        before = 0;
        for (uint64_t u = threadIdx.x; u <= L.n; u += kPackBlock) loff[u] = 0;
        return;
    }
#pragma unroll 4
    for (uint64_t u = threadIdx.x; u <= L.n; u += kPackBlock) {
        const uint32_t o = L.off[u];
        const uint32_t x = o >> 6;
        const uint32_t first = o < L.m ? rank[x] + (uint32_t)__popcll(bits[x] & ((1ull << (o & 63u)) - 1ull)) : before;
        loff[u] = first | (u < L.n && L.off[u + 1] > o ? kHasArcs : 0u);
    }
}

// One trial's arcs as a cascade walks them: packed (its live graph), or the
// graph's own arcs with the trial's coin bits.
struct LiveGraph {
    const uint32_t* __restrict__ off;
    const uint32_t* __restrict__ to;
    const uint64_t* __restrict__ bits;
    const uint64_t* __restrict__ rec;
};

template <bool kPacked>
__device__ __forceinline__ LiveGraph live_graph(const LiveParams& L, uint32_t row)
{
    if constexpr (kPacked) return LiveGraph{L.loff + (uint64_t)row * (L.n + 1), L.llist + (uint64_t)row * L.list_cap, nullptr, nullptr};
    else return LiveGraph{L.off, L.idx, L.rows + (uint64_t)row * L.row_words, L.rec};
}

// Small cascades: lane = one (trial, set), which follows its cascade alone
// over a list of at most kTinyCap nodes; a cascade that outgrows the list is
// put on the trial's work list for live_reach_kernel.  Most cascades of single
// nodes end here without taking a wavefront.  Workgroup b serves the trials of
// XCD b % 8, so a trial's live graph is read by one L2.
template <bool kPacked>
__global__ __launch_bounds__(kBlock) void live_tiny_kernel(LiveParams L)
{
    __shared__ uint32_t lists[kWaves][kTinyCap][64];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t q = blockIdx.x % kLiveQueues;
    const uint32_t groups = (L.n_sets + kBlock - 1) / kBlock;
    const uint32_t k = blockIdx.x / kLiveQueues;
    const uint32_t row = (k / groups) * kLiveQueues + q;
    const uint32_t set = (k % groups) * kBlock + threadIdx.x;
    if (row >= L.tc) return;
    uint32_t(&list)[kTinyCap][64] = lists[threadIdx.x >> 6];
    const LiveGraph G = live_graph<kPacked>(L, row);
    const uint64_t bm_words = 2 * ((L.n + 63) / 64);
    const uint32_t* base = L.base ? L.base + (uint64_t)row * bm_words : nullptr;
    bool big = false;
    uint32_t cnt = 0, depth = 0;
    if (set < L.n_sets) {
        const uint32_t s0 = L.set_off[set], ns = L.set_off[set + 1] - s0;
        big = ns > kTinySeeds;
        for (uint32_t i = 0; i < ns && !big; ++i) {
            const uint32_t v = L.set_nodes[s0 + i];
            if (!base || !((base[v >> 5] >> (v & 31u)) & 1u)) list[cnt++][lane] = v;
        }
        // level by level: [head, end) is the current level
        uint32_t head = 0, end = cnt;
        bool arcs = false;
        while (head < cnt && !big) {
            const uint32_t u = list[head][lane];
            uint2 r;
            __builtin_memcpy(&r, G.off + u, sizeof r);
            auto meet = [&](uint32_t v) {
                if (base && ((base[v >> 5] >> (v & 31u)) & 1u)) return;
                bool seen = false;
                for (uint32_t i = 0; i < cnt; ++i) seen |= list[i][lane] == v;
                if (seen) return;
                if (cnt == kTinyCap) big = true;
                else list[cnt++][lane] = v;
            };
            if constexpr (kPacked) {
                arcs |= (r.x & kHasArcs) != 0;
                r.x &= ~kHasArcs;
                r.y &= ~kHasArcs;
                for (uint32_t k = r.x; k < r.y && !big; ++k) meet(G.to[k]);
            } else {
                arcs |= r.y > r.x;
                if (r.y - r.x > kTinyDeg) {
                    big = true;
                    break;
                }
                for (uint32_t x = r.x >> 6; r.y > r.x && x <= (r.y - 1) >> 6 && !big; ++x) {
                    uint64_t b = G.bits[x] & range_of(r.x > 64 * x ? r.x - 64 * x : 0u, r.y - 64 * x < 64u ? r.y - 64 * x : 64u);
                    for (; b && !big; b &= b - 1) meet(G.to[64 * x + (uint32_t)__builtin_ctzll(b)]);
                }
            }
            if (++head == end) {
                if (arcs) ++depth;
                arcs = false;
                end = cnt;
            }
        }
        if (!big) {
            if (cnt) atomicAdd((unsigned long long*)&L.totals[set], (unsigned long long)cnt);
            if (L.set_node_counts)
                for (uint32_t i = 0; i < cnt; ++i) atomicAdd(&L.set_node_counts[(uint64_t)set * L.n + list[i][lane]], 1u);
        }
    }
    const uint64_t bigs = __ballot(big);
    if (bigs) {
        uint32_t at = 0;
        if (lane == 0) {
            at = atomicAdd(&L.todo_count[row], (uint32_t)__popcll(bigs));
            atomicAdd(&L.entries[kCtlStep * q], (uint32_t)__popcll(bigs));
        }
        at = uniform32(at);
        if (big) L.todo[(uint64_t)row * L.n_sets + at + lanes_below(bigs)] = set;
        depth = big ? 0u : depth;
    }
    // the largest step count of the wavefront
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t y = (uint32_t)__shfl_xor((int)depth, o);
        depth = y > depth ? y : depth;
    }
    if (lane == 0 && depth > load_relaxed32(&L.status[0])) atomicMax(&L.status[0], depth);
}

// Workgroup-wide state of one cascade.
template <int kW>
struct LiveShared {
    uint32_t buf[kW][kLiveBuf];  // live arcs waiting for their targets, per wavefront
    uint64_t q[2][kLiveQ];       // first entries of the current and the next level (packed: nodes, else arc records)
    uint32_t cnt;                // nodes of the next level
    uint32_t arcs;               // the level holds a node with out-arcs
    uint32_t task, n_tasks;
};

// One cascade of a trial: nodes reached over its live graph from the nodes
// that `seed_at(i)` names, level by level.  bm: visited bitmap in LDS; list:
// the nodes in the order reached (each level consecutive).  Per round a
// wavefront takes 64 nodes of the level (lane = node) and reads their live
// bounds; their live arcs are laid out densely in LDS (a prefix sum of the
// counts) so that the targets are fetched 64 at a time, tested and set in the
// bitmap and appended.  `level(l, count)` is told the size of every level.
// Bound by the latency of the two dependent reads per round (bounds, target;
// coin words, target record).  Once all n nodes are reached, the arcs left
// lead nowhere new and are not walked.  Returns the node count; steps = levels
// holding a node with out-arcs.
template <int kW, bool kPacked, typename SeedAt, typename Level>
__device__ __forceinline__ uint32_t live_cascade(const LiveGraph& G, uint32_t n, uint32_t* bm, uint32_t* list,
                                                 LiveShared<kW>& sh, uint32_t n_seeds, SeedAt seed_at, Level level, uint32_t& steps)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = kW == 1 ? 0u : uniform32(threadIdx.x >> 6);
    uint32_t* buf = sh.buf[wave];
    // what an arc leads to: a node, or its record
    using To = typename std::conditional<kPacked, uint32_t, uint64_t>::type;
    auto node_of = [](To x) -> uint32_t { return kPacked ? (uint32_t)x : rec_node(x); };
    auto fetch = [&](uint32_t e) -> To {
        if constexpr (kPacked) return G.to[e];
        else return G.rec[e];
    };
    uint32_t par = 0;           // q[par] holds the level being filled
    uint32_t hi = 0, fill = 0;  // list entries below hi are final; fill: entries of the level being filled (one wavefront)
    // visit v[y] of lane where 64 y + lane < nn: the bitmap updates are issued
    // together, then the new nodes of all slots take their places at once
    auto visit = [&](uint32_t nn, const To (&v)[kLiveBuf / 64]) {
        bool fresh[kLiveBuf / 64];
        wait_loads();
#pragma unroll
        for (uint32_t y = 0; y < kLiveBuf / 64; ++y) {
            fresh[y] = false;
            if (64 * y >= nn) continue;
            const uint32_t u = node_of(v[y]), bit = 1u << (u & 31u);
            fresh[y] = 64 * y + lane < nn && (atomicOr(&bm[u >> 5], bit) & bit) == 0;
        }
        uint64_t mask[kLiveBuf / 64];
        uint32_t k = 0;
#pragma unroll
        for (uint32_t y = 0; y < kLiveBuf / 64; ++y) {
            mask[y] = 0;
            if (64 * y >= nn) continue;
            mask[y] = __ballot(fresh[y]);
            k += (uint32_t)__popcll(mask[y]);
        }
        if (k == 0) return;
        uint32_t at;
        if constexpr (kW == 1) {
            at = fill;
            fill += k;
        } else {
            at = 0;
            if (lane == 0) at = atomicAdd(&sh.cnt, k);
            at = uniform32(at);
        }
#pragma unroll
        for (uint32_t y = 0; y < kLiveBuf / 64; ++y) {
            if (64 * y >= nn) break;
            if (fresh[y]) {
                const uint32_t pos = at + lanes_below(mask[y]);
                list[hi + pos] = node_of(v[y]);
                if (pos < kLiveQ) sh.q[par][pos] = v[y];
            }
            at += (uint32_t)__popcll(mask[y]);
        }
    };
    if (kW > 1 && threadIdx.x == 0) {
        sh.cnt = 0;
        sh.arcs = 0;
    }
    __syncthreads();
    for (uint32_t i = 64 * wave; i < n_seeds; i += 64 * kW) {
        To v[kLiveBuf / 64] = {};
        if (i + lane < n_seeds) {
            const uint32_t u = seed_at(i + lane);
            if constexpr (kPacked) v[0] = u;
            else v[0] = arc_record(u, G.off[u], G.off[u + 1]);
        }
        visit(n_seeds - i < 64 ? n_seeds - i : 64u, v);
    }
    steps = 0;
    uint32_t lev = 0, lo = 0;
    for (;;) {
        __syncthreads();
        if constexpr (kW > 1) fill = sh.cnt;
        const uint32_t count = fill;
        if (count == 0) break;
        level(lev, count);
        ++lev;
        lo = hi;
        hi += count;
        par ^= 1u;
        fill = 0;
        bool any = false;
        if constexpr (kW > 1) {
            __syncthreads();
            if (threadIdx.x == 0) {
                sh.cnt = 0;
                sh.arcs = 0;
            }
            __syncthreads();
        }
        for (uint32_t i = 64 * wave; i < count; i += 64 * kW) {
            const bool have = i + lane < count;
            // the node's bounds: from its record, or (packed, and entries
            // beyond the LDS) both in one 8-byte read
            uint2 r = make_uint2(0u, 0u);
            if (have) {
                const bool near = i + lane < kLiveQ;
                const uint64_t x = near ? sh.q[par ^ 1u][i + lane] : (uint64_t)list[lo + i + lane];
                if (!kPacked && near) r = make_uint2(rec_first(x), rec_first(x) + rec_degree(x));
                else __builtin_memcpy(&r, G.off + (uint32_t)x, sizeof r);
            }
            const bool all = hi + (kW == 1 ? fill : uniform32(*(volatile uint32_t*)&sh.cnt)) >= n;
            // fetch and visit the targets of buf[0 .. nn)
            auto visit_buf = [&](uint32_t nn) {
                To v[kLiveBuf / 64];
#pragma unroll
                for (uint32_t y = 0; y < kLiveBuf / 64; ++y) v[y] = 64 * y + lane < nn ? fetch(buf[64 * y + lane]) : 0u;
                visit(nn, v);
            };
            if constexpr (kPacked) {
                any |= __ballot((r.x & kHasArcs) != 0) != 0;
                if (all && any) break;
                if (all) continue;
                const uint32_t k0 = r.x & ~kHasArcs;
                const uint32_t deg = (r.y & ~kHasArcs) - k0;
                const uint32_t c = deg <= kLaneArcs ? deg : 0u;
                const uint32_t incl = wave_scan_incl(c);
                const uint32_t total = uniform32((uint32_t)__builtin_amdgcn_readlane((int)incl, 63));
                for (uint32_t win = 0; win < total; win += kLiveBuf) {
                    const uint32_t p = incl - c - win;  // wraps below the window
                    __builtin_amdgcn_wave_barrier();
                    for (uint32_t k = 0; k < c; ++k)
                        if (p + k < kLiveBuf) buf[p + k] = k0 + k;
                    __builtin_amdgcn_wave_barrier();
                    visit_buf(total - win < kLiveBuf ? total - win : kLiveBuf);
                }
                uint64_t longs = __ballot(deg > kLaneArcs);
                while (longs) {
                    const int j = __builtin_ctzll(longs);
                    longs &= longs - 1;
                    const uint32_t a0 = (uint32_t)__builtin_amdgcn_readlane((int)k0, j);
                    const uint32_t a1 = a0 + (uint32_t)__builtin_amdgcn_readlane((int)deg, j);
                    for (uint32_t k = a0; k < a1; k += kLiveBuf) {
                        To v[kLiveBuf / 64];
#pragma unroll
                        for (uint32_t y = 0; y < kLiveBuf / 64; ++y) v[y] = k + 64 * y + lane < a1 ? fetch(k + 64 * y + lane) : 0u;
                        visit(a1 - k < kLiveBuf ? a1 - k : kLiveBuf, v);
                    }
                }
            } else {
                const uint32_t o0 = r.x, o1 = r.y;
                const uint32_t x0 = o0 >> 6;
                const uint32_t nw = o1 > o0 ? ((o1 - 1) >> 6) - x0 + 1 : 0u;  // coin words of the row
                any |= __ballot(nw != 0) != 0;
                if (all && any) break;
                if (all) continue;
                // lay the set bits of up to two words per lane out in LDS and visit their targets
                auto walk = [&](const uint64_t (&word)[2], uint32_t ebase) {
                    const uint32_t c = (uint32_t)(__popcll(word[0]) + __popcll(word[1]));
                    const uint32_t incl = wave_scan_incl(c);
                    const uint32_t total = uniform32((uint32_t)__builtin_amdgcn_readlane((int)incl, 63));
                    for (uint32_t win = 0; win < total; win += kLiveBuf) {
                        uint32_t p = incl - c - win;  // wraps below the window
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (uint32_t y = 0; y < 2; ++y)
                            for (uint64_t b = word[y]; b; b &= b - 1, ++p)
                                if (p < kLiveBuf) buf[p] = ebase + 64 * y + (uint32_t)__builtin_ctzll(b);
                        __builtin_amdgcn_wave_barrier();
                        visit_buf(total - win < kLiveBuf ? total - win : kLiveBuf);
                    }
                };
                uint64_t word[2];
#pragma unroll
                for (uint32_t y = 0; y < 2; ++y) word[y] = nw <= 2 && y < nw ? G.bits[x0 + y] : 0ull;
                if (nw && nw <= 2) {
                    word[0] &= ~0ull << (o0 & 63u);
                    const uint64_t tail = ~0ull >> (63u - ((o1 - 1) & 63u));
                    if (nw == 1) word[0] &= tail;
                    else word[1] &= tail;
                }
                walk(word, 64 * x0);
                // long rows: lane = two consecutive words of the row
                uint64_t longs = __ballot(nw > 2);
                while (longs) {
                    const int j = __builtin_ctzll(longs);
                    longs &= longs - 1;
                    const uint32_t a0 = (uint32_t)__builtin_amdgcn_readlane((int)o0, j), a1 = (uint32_t)__builtin_amdgcn_readlane((int)o1, j);
                    const uint32_t y1 = (a1 - 1) >> 6;
                    for (uint32_t y0 = a0 >> 6; y0 <= y1; y0 += 128) {
#pragma unroll
                        for (uint32_t y = 0; y < 2; ++y) {
                            const uint32_t x = y0 + 2 * lane + y;
                            word[y] = x <= y1 ? G.bits[x] : 0ull;
                            if (x == a0 >> 6) word[y] &= ~0ull << (a0 & 63u);
                            if (x == y1) word[y] &= ~0ull >> (63u - ((a1 - 1) & 63u));
                        }
                        walk(word, 64 * (y0 + 2 * lane));
                    }
                }
            }
        }
        if constexpr (kW > 1) {
            if (any && lane == 0) sh.arcs = 1;
            __syncthreads();
            any = sh.arcs != 0;
        }
        if (any) ++steps;
    }
    return hi;
}

// The listed (trial, set) cascades, kW wavefronts each.  Workgroups take
// entries from their XCD's queue in row order, so that an XCD's workgroups
// read few trials' live graphs at a time (they stay in its L2), then from the
// others'.  Bitmaps are clear (or hold the trial's base) between cascades: a
// cascade clears what it set.
template <int kW, bool kPacked>
__global__ __launch_bounds__(64 * kW) void live_reach_kernel(LiveParams L)
{
    extern __shared__ uint32_t bm[];  // [2 * ceil(n / 64)]
    __shared__ LiveShared<kW> sh;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t bm_words = (uint32_t)(2 * ((L.n + 63) / 64));
    uint32_t* list = L.queue + (uint64_t)blockIdx.x * L.n;
    for (uint32_t i = threadIdx.x; i < bm_words; i += 64 * kW) bm[i] = 0;
    uint32_t held = ~0u;  // row whose base the bitmap holds
    uint32_t max_steps = 0;
    for (uint32_t turn = 0; turn < kLiveQueues; ++turn) {
        const uint32_t q = (blockIdx.x + turn) % kLiveQueues;
        uint32_t* taken = &L.taken[kCtlStep * q];
        const uint32_t entries = L.entries[kCtlStep * q];
        if (entries == 0) continue;
        // a window of 64 of the queue's rows: entries up to and with lane's row
        uint32_t i0 = 0, incl = 0, before = 0, total = 0;
        auto window = [&]() {
            const uint32_t r = q + kLiveQueues * (i0 + lane);
            incl = wave_scan_incl(r < L.tc ? L.todo_count[r] : 0u);
            total = uniform32((uint32_t)__builtin_amdgcn_readlane((int)incl, 63));
        };
        window();
        for (;;) {
            __syncthreads();
            // (a drained queue is seen by a plain read: thousands of
            // workgroups adding to one counter take 0.2 ms)
            if (threadIdx.x == 0) sh.task = load_relaxed32(taken) < entries ? atomicAdd(taken, L.take) : entries;
            __syncthreads();
            const uint32_t first = uniform32(sh.task);
            if (first >= entries) break;
            for (uint32_t k = first; k < entries && k < first + L.take; ++k) {
                // (k < entries = the sum of the queue's row counts, so a window holds it)
                while (k - before >= total) {
                    before += total;
                    i0 += 64;
                    window();
                }
                const uint32_t j = (uint32_t)__builtin_ctzll(__ballot(incl > k - before));
                const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)incl, (int)j);
                const uint32_t row = q + kLiveQueues * (i0 + j);
                const uint32_t set = uniform32(L.todo[(uint64_t)row * L.n_sets + (L.todo_count[row] - (end - (k - before)))]);
                const uint32_t* base = L.base ? L.base + (uint64_t)row * bm_words : nullptr;
                if (base && held != row) {
                    __syncthreads();
                    for (uint32_t i = threadIdx.x; i < bm_words; i += 64 * kW) bm[i] = base[i];
                    held = row;
                }
                const uint32_t s0 = L.set_off[set];
                uint32_t steps;
                const uint32_t cnt = live_cascade<kW, kPacked>(
                    live_graph<kPacked>(L, row), (uint32_t)L.n, bm, list, sh, L.set_off[set + 1] - s0,
                    [&](uint32_t i) { return L.set_nodes[s0 + i]; }, [](uint32_t, uint32_t) {}, steps);
                max_steps = steps > max_steps ? steps : max_steps;
                if (threadIdx.x == 0 && cnt) atomicAdd((unsigned long long*)&L.totals[set], (unsigned long long)cnt);
                if (L.set_node_counts)
                    for (uint32_t i = threadIdx.x; i < cnt; i += 64 * kW) atomicAdd(&L.set_node_counts[(uint64_t)set * L.n + list[i]], 1u);
                if (cnt > bm_words) {
                    for (uint32_t i = threadIdx.x; i < bm_words; i += 64 * kW) bm[i] = base ? base[i] : 0u;
                } else {
                    for (uint32_t i = threadIdx.x; i < cnt; i += 64 * kW) {
                        const uint32_t v = list[i];
                        if (base) atomicAnd(&bm[v >> 5], ~(1u << (v & 31u)));
                        else bm[v >> 5] = 0;
                    }
                }
            }
        }
    }
    if (threadIdx.x == 0 && max_steps) atomicMax(&L.status[0], max_steps);
}

// Seeds of a single-set run, passed with the launch when they fit.
constexpr uint32_t kArgSeeds = 256;  // (a workgroup of kBlock threads places them)
static_assert(kArgSeeds <= kBlock);
struct LiveSeeds {
    uint32_t count;
    const uint32_t* more;  // the seeds in device memory when there are more than kArgSeeds, else null
    uint32_t v[kArgSeeds];
};

// What a slot run reads, put in place by one launch: its item, its seeds, its
// cleared outputs (uploads and fills of their own took 30 us a run).
__global__ __launch_bounds__(kBlock) void slot_prologue_kernel(BatchItem it, LiveSeeds S, BatchItem* __restrict__ item, uint32_t* __restrict__ seeds,
                                                               uint32_t* __restrict__ status)
{
    const uint64_t i0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x, step = (uint64_t)gridDim.x * kBlock;
    for (uint64_t t = i0; t < it.P.T; t += step) it.trial_counts[t] = 0;
    if (it.node_counts)
        for (uint64_t v = i0; v < (uint64_t)it.P.n; v += step) it.node_counts[v] = 0;
    if (blockIdx.x != 0) return;
    if (threadIdx.x < S.count) seeds[threadIdx.x] = S.v[threadIdx.x];
    if (threadIdx.x < 4) status[threadIdx.x] = 0;
    if (threadIdx.x == 4) *it.total = 0;
    if (threadIdx.x == 5) *item = it;
}

// One seed set over every trial of a range: workgroups run the trials t0 + b,
// t0 + b + gridDim.x, ... over their coin rows and leave the final bitmaps for
// live_nodes_kernel.
template <int kW>
__global__ __launch_bounds__(64 * kW) void live_single_kernel(LiveParams L, LiveSeeds S, uint32_t* __restrict__ bitmaps,
                                                             uint32_t* __restrict__ trial_counts, uint64_t* __restrict__ total,
                                                             uint32_t* __restrict__ level_counts, uint32_t max_levels)
{
    extern __shared__ uint32_t bm[];  // [2 * ceil(n / 64)]
    __shared__ LiveShared<kW> sh;
    const uint32_t bm_words = (uint32_t)(2 * ((L.n + 63) / 64));
    uint64_t sum = 0;
    uint32_t max_steps = 0;
    for (uint32_t row = blockIdx.x; row < L.tc; row += gridDim.x) {
        const uint32_t t = L.t0 + row;
        for (uint32_t i = threadIdx.x; i < bm_words; i += 64 * kW) bm[i] = 0;
        uint32_t steps;
        const uint32_t cnt = live_cascade<kW, false>(
            live_graph<false>(L, row), (uint32_t)L.n, bm, L.queue + (uint64_t)blockIdx.x * L.n, sh, S.count,
            [&](uint32_t i) { return S.more ? S.more[i] : S.v[i]; },
            [&](uint32_t l, uint32_t count) {
                if (level_counts && threadIdx.x == 0 && l < max_levels) level_counts[(uint64_t)l * L.T + t] = count;
            },
            steps);
        if (bitmaps)
            for (uint32_t i = threadIdx.x; i < bm_words; i += 64 * kW) bitmaps[(uint64_t)row * bm_words + i] = bm[i];
        if (threadIdx.x == 0) trial_counts[t] = cnt;
        sum += cnt;
        max_steps = steps > max_steps ? steps : max_steps;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (sum) atomicAdd((unsigned long long*)total, (unsigned long long)sum);
        if (max_steps > load_relaxed32(&L.status[0])) atomicMax(&L.status[0], max_steps);
    }
}

// Per-node counts and word-major bits from the trials' bitmaps: a workgroup
// takes 64 nodes and kNodeWords words of 64 trials, a wavefront every
// kWaves-th of them (lane = trial, then, transposed, lane = node).
// node_counts were cleared by the draw of the first range.
constexpr uint32_t kNodeWords = 16;
__global__ __launch_bounds__(kBlock) void live_nodes_kernel(const uint32_t* __restrict__ bitmaps, uint64_t bm_words, uint64_t n, uint32_t t0,
                                                            uint32_t tc, uint32_t* __restrict__ node_counts, uint64_t* __restrict__ A)
{
    __shared__ uint32_t part[kWaves][64];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint64_t tile = blockIdx.x;
    const uint64_t v = tile * 64 + lane;
    uint32_t c = 0;
#pragma unroll
    for (uint32_t k = 0; k < kNodeWords / kWaves; ++k) {
        const uint32_t w = blockIdx.y * kNodeWords + kWaves * k + wave;
        const uint32_t row = 64 * w + lane;
        uint64_t x = row < tc ? *reinterpret_cast<const uint64_t*>(bitmaps + (uint64_t)row * bm_words + 2 * tile) : 0ull;
        x = wave_transpose64(x, lane);
        c += (uint32_t)__popcll(x);
        if (A && v < n && 64 * w < tc) A[((uint64_t)t0 / 64 + w) * n + v] = x;
    }
    part[wave][lane] = c;
    __syncthreads();
    if (wave == 0 && v < n && node_counts) {
#pragma unroll
        for (int q = 1; q < kWaves; ++q) c += part[q][lane];
        if (c) atomicAdd(&node_counts[v], c);
    }
}

}  // namespace imsim
