// Kernels of the per-trial push form: one small workgroup runs one trial's
// whole cascade by pushing, for LT with every node's distance to its threshold
// in LDS or, on larger graphs, in a row of device memory, for IC (kBits = 1)
// with the active nodes in LDS and each arc's coin drawn as the arc is met.
//
// Section 2's LT rule (v joins when the weight of its active in-neighbours
// exceeds its threshold) needs, per node and trial, one number that every
// newly active in-neighbour lowers once; the trial joins v in the step that
// takes it past zero.  A grid-wide sweep re-reads all in-neighbours of every
// pending node at every step, and a cascade on a sparse graph takes hundreds
// of steps, each a launch; here a step is one round of a workgroup and every
// arc is touched once.  The fixpoint does not depend on the order.
#pragma once

#include "live_kernels.hpp"

namespace imsim {

constexpr uint32_t kLtRing = 256;  // most recent joins kept in LDS (older ones are read back from the list)

// Per (node, trial) state by element width:
//  8, 16: equal in-weights; 2^(bits-1) - k plus the active in-arcs so far, k
//         the least number of them that joins the node; the top bit is the
//         node's active bit, and sums cannot pass the element (in-arcs < 2^(bits-1) - 1)
//  32:    threshold minus the active in-weight so far, modulo 2^32: in-weights
//         sum to at most 2^32, so "weight > remainder" holds at the crossing
//         and never again; active bits in a bitmap of their own
//  1:     IC, the coin of an out-arc drawn when its source has joined; the
//         bitmap alone
struct LtRun {
    uint64_t n;
    const uint32_t* __restrict__ off;  // [n + 1] out-CSR offsets
    const uint64_t* __restrict__ rec;     // [m] arc records
    const uint64_t* __restrict__ wout;    // weight per out-arc (32-bit elements)
    const int64_t* __restrict__ in_off;   // in-CSR, equal in-weights: pieces per node
    const uint32_t* __restrict__ in_src;  // their sources
    const uint32_t* __restrict__ node_w;  // and their weight
    const uint32_t* __restrict__ thr;     // IC: threshold per out-arc
    uint32_t* node_counts;                // IC: [n] counted as nodes join, or null
    uint8_t* rows;      // [tc][stride] starting states
    uint64_t stride;    // bytes, a multiple of 16
    uint64_t seed;
    uint32_t t0, tc;    // trials of this range
    uint32_t* queue;    // [workgroup][n] nodes in the order they joined
    uint32_t* bitmaps;  // [tc][2 * ceil(n / 64)] final active nodes, or null
    uint32_t* trial_counts;
    uint64_t* total;
    uint32_t* status;
};

// Starting states: lane = node, one 64-trial word per wavefront (the hash
// rounds that do not depend on the trials are shared by a node's blocks).
template <int kBits>
__global__ __launch_bounds__(kBlock) void lt_rows_kernel(LiveClear C, LtRun R)
{
    const uint32_t lane = threadIdx.x & 63u;
    if (C.total) {
        if (C.status && blockIdx.x == 0 && threadIdx.x < 4) C.status[threadIdx.x] = 0;
        if (blockIdx.x == 0 && threadIdx.x == 4) *C.total = 0;
        if (C.node_counts)
            for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v < C.n; v += (uint64_t)gridDim.x * kBlock) C.node_counts[v] = 0;
    }
    const uint64_t wave = uniform64(((uint64_t)blockIdx.x * kBlock + threadIdx.x) >> 6);
    const uint64_t tiles = (R.n + 63) / 64;
    const uint64_t words = (R.tc + 63) / 64;
    if (wave >= tiles * words) return;
    const uint64_t w = wave / tiles, v = (wave - w * tiles) * 64 + lane;
    const uint32_t left = R.tc - (uint32_t)(64 * w);
    const uint32_t groups = left >= 64 ? 8u : (left + 7) / 8;
    constexpr uint32_t kHalf = kBits == 32 ? 0u : 1u << (kBits - 1);
    uint32_t wv = 0, inv = 0;
    bool one = false;  // a single in-arc of weight 2^32 (stored as two pieces): its source joins the node
    if (kBits != 32 && v < R.n) {
        wv = R.node_w[v];
        inv = wv >= 2 ? (uint32_t)(0x100000000ull / wv) : 0u;
        const int64_t k0 = R.in_off[v];
        one = wv == 1u << 31 && R.in_off[v + 1] - k0 == 2 && R.in_src[k0] == R.in_src[k0 + 1];
    }
    const PhiloxArc a = philox_arc(v, R.seed, kDomainLtNode);
    uint8_t* out = R.rows + 64 * w * R.stride + v * (kBits / 8);
    for (uint32_t g = 0; g < groups; ++g) {
        const Block4 b = philox_group(a, R.t0 / 8 + 8 * w + g, R.seed, kDomainLtNode);
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) {
            const uint32_t h = block_lane(b, j);
            uint8_t* at = out + (uint64_t)(8 * g + j) * R.stride;
            if (v < R.n && 8 * g + j < left) {
                if constexpr (kBits == 32) *reinterpret_cast<uint32_t*>(at) = h;
                else {
                    const uint32_t start = kHalf - (one ? 1u : kmin_of(h, wv, inv, kHalf - 1));
                    if constexpr (kBits == 8) *at = (uint8_t)start;
                    else *reinterpret_cast<uint16_t*>(at) = (uint16_t)start;
                }
            }
        }
    }
}

// Zeroes a run's outputs (the IC runs here have no earlier kernel to do it).
__global__ __launch_bounds__(kBlock) void trial_clear_kernel(LiveClear C)
{
    if (C.status && blockIdx.x == 0 && threadIdx.x < 4) C.status[threadIdx.x] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 4) *C.total = 0;
    if (C.node_counts)
        for (uint64_t v = (uint64_t)blockIdx.x * kBlock + threadIdx.x; v < C.n; v += (uint64_t)gridDim.x * kBlock) C.node_counts[v] = 0;
}

template <int kW>
struct LtTrialShared {
    uint32_t buf[kW][kLiveBuf];  // out-arcs waiting for their targets, per wavefront
    uint64_t ring[kLtRing];      // the record of join number i at i % kLtRing
    uint32_t tail;               // joins so far
};

// Trials t0 + b, t0 + b + gridDim.x, ... of one run, kW wavefronts each, the
// trial's state in LDS (kLds) or in its row where it stands.  A
// round takes up to 64 * kW joined nodes (lane = node), lays their out-arcs
// out densely in LDS (a prefix sum of the degrees), fetches 64 targets at a
// time and updates their states.  Bound by the chain of rounds: one dependent
// read (the target records, which bring the next round's row bounds) and the
// update.
template <int kBits, int kW, bool kLds>
__global__ __launch_bounds__(64 * kW) void lt_trial_kernel(LtRun R, LiveSeeds S)
{
    extern __shared__ uint32_t lds[];  // state, then (32-bit elements) the active bitmap
    __shared__ LtTrialShared<kW> sh;
    constexpr uint32_t kHalf = kBits == 32 ? 0u : 1u << (kBits - 1);
    constexpr uint32_t kPer = 32 / kBits;  // elements per LDS word
    constexpr bool kIc = kBits == 1;
    static_assert(!kIc || kLds, "the IC bitmap is in LDS");
    constexpr uint32_t kSlots = kLiveBuf / 64;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = kW == 1 ? 0u : uniform32(threadIdx.x >> 6);
    const uint32_t n = (uint32_t)R.n;
    const uint32_t bm_words = 2 * ((n + 63) / 64);
    const uint32_t st_words = kIc ? 0u : (uint32_t)(R.stride / 4);
    uint32_t* buf = sh.buf[wave];
    uint32_t* list = R.queue + (uint64_t)blockIdx.x * R.n;
    uint64_t sum = 0;
    uint32_t max_rounds = 0;
    for (uint32_t row = blockIdx.x; row < R.tc; row += gridDim.x) {
        uint32_t* const start = reinterpret_cast<uint32_t*>(R.rows + (uint64_t)row * R.stride);
        uint32_t* const st = kLds ? lds : start;
        uint32_t* const bm = kLds ? lds + st_words : R.bitmaps + (uint64_t)row * bm_words;
        if constexpr (kLds && !kIc)
            for (uint32_t i = threadIdx.x; i < st_words / 4; i += 64 * kW)
                reinterpret_cast<uint4*>(lds)[i] = reinterpret_cast<const uint4*>(start)[i];
        if (kBits == 32 || kIc)
            for (uint32_t i = threadIdx.x; i < bm_words; i += 64 * kW) bm[i] = 0;
        if (kW > 1 && threadIdx.x == 0) sh.tail = 0;
        __syncthreads();
        uint32_t tail = 0, head = 0, rounds = 0;
        uint32_t level_end = 0;       // IC: rounds stay within a level (steps are counted by levels)
        uint32_t level = 0;           // IC: levels begun; rounds = the last one holding a node with out-arcs
        uint32_t seen = 0, kept = 0;  // joins of the rounds behind; the ring holds none before `kept`
        // v[y] of every lane with fresh[y] joined
        auto append = [&](const bool (&fresh)[kSlots], const uint64_t (&v)[kSlots]) {
            uint64_t mask[kSlots];
            uint32_t k = 0;
#pragma unroll
            for (uint32_t y = 0; y < kSlots; ++y) {
                mask[y] = __ballot(fresh[y]);
                k += (uint32_t)__popcll(mask[y]);
            }
            if (k == 0) return;
            uint32_t at;
            if constexpr (kW == 1) {
                at = tail;
                tail += k;
            } else {
                at = 0;
                if (lane == 0) at = atomicAdd(&sh.tail, k);
                at = uniform32(at);
            }
#pragma unroll
            for (uint32_t y = 0; y < kSlots; ++y) {
                if (fresh[y]) {
                    const uint32_t pos = at + lanes_below(mask[y]);
                    const uint32_t u = rec_node(v[y]);
                    list[pos] = u;
                    sh.ring[pos % kLtRing] = v[y];
                    if (kIc && R.node_counts) atomicAdd(&R.node_counts[u], 1u);
                }
                at += (uint32_t)__popcll(mask[y]);
            }
        };
        // a newly active in-neighbour of weight wt: does it take v past its threshold
        // (IC: wt is arc e's threshold, and its coin decides)
        const uint32_t t = R.t0 + row;
        auto crosses = [&](uint32_t v, uint64_t wt, uint32_t e) {
            if constexpr (kIc) {
                const uint32_t th = (uint32_t)wt;
                if (th == 0) return false;
                if (th != 0xFFFFFFFFu) {
                    const Block4 b = philox_block_chain(e, t >> 3, R.seed, kDomainIcArc);
                    if (block_lane(b, t & 7u) >= th) return false;
                }
                const uint32_t bit = 1u << (v & 31u);
                return (atomicOr(&bm[v >> 5], bit) & bit) == 0;
            } else if constexpr (kBits == 32) {
                if (wt == 0 || wt <= atomicSub(&st[v], (uint32_t)wt)) return false;
                const uint32_t bit = 1u << (v & 31u);
                return (atomicOr(&bm[v >> 5], bit) & bit) == 0;  // (seeds cross too)
            } else {
                const uint32_t shift = (v % kPer) * kBits;
                const uint32_t old = atomicAdd(&st[v / kPer], 1u << shift) >> shift;
                return (old & (2 * kHalf - 1)) == kHalf - 1;
            }
        };
        for (uint32_t i = 64 * wave; i < S.count; i += 64 * kW) {
            bool on[kSlots] = {};
            uint64_t vs[kSlots] = {};
            on[0] = i + lane < S.count;
            if (on[0]) {
                const uint32_t v = S.more ? S.more[i + lane] : S.v[i + lane];
                vs[0] = arc_record(v, R.off[v], R.off[v + 1]);
                if constexpr (kBits == 32 || kIc) {
                    atomicOr(&bm[v >> 5], 1u << (v & 31u));
                } else {
                    const uint32_t shift = (v % kPer) * kBits;
                    atomicAnd(&st[v / kPer], ~((2 * kHalf - 1) << shift));
                    atomicOr(&st[v / kPer], kHalf << shift);
                }
            }
            append(on, vs);
        }
        for (;;) {
            __syncthreads();
            if constexpr (kW > 1) tail = sh.tail;
            if (head >= tail) break;
            // joins of one round land in the ring in no order between the
            // wavefronts, so a round of more than the ring holds leaves it unusable
            if (kW > 1 && tail - seen > kLtRing) kept = tail;
            seen = tail;
            if (kIc && head == level_end) {
                level_end = tail;
                ++level;
            }
            const uint32_t stop = kIc ? level_end : tail;
            const uint32_t end = stop - head < 64 * kW ? stop : head + 64 * kW;
            const uint32_t i = head + 64 * wave + lane;
            const bool have = i < end;
            uint32_t o0 = 0, deg = 0;
            if (have) {
                if (tail - i <= kLtRing && i >= kept) {
                    const uint64_t x = sh.ring[i % kLtRing];
                    o0 = rec_first(x);
                    deg = rec_degree(x);
                } else {
                    uint2 r;
                    __builtin_memcpy(&r, R.off + list[i], sizeof r);
                    o0 = r.x;
                    deg = r.y - r.x;
                }
            }
            head = end;
            if (!kIc) ++rounds;
            if constexpr (kW > 1) __syncthreads();  // every entry is read before the ring moves on
            if (kIc && __ballot(deg != 0)) rounds = level;  // (of this wavefront's nodes)
            const uint32_t c = deg <= kLaneArcs ? deg : 0u;
            const uint32_t incl = wave_scan_incl(c);
            const uint32_t total = uniform32((uint32_t)__builtin_amdgcn_readlane((int)incl, 63));
            auto visit_arcs = [&](auto arc_at, uint32_t nn) {
                // loads, updates and appends of all slots each go together
                uint64_t v[kSlots];
                uint64_t wt[kSlots];
                uint32_t e[kSlots];
                bool fresh[kSlots];
#pragma unroll
                for (uint32_t y = 0; y < kSlots; ++y) {
                    const bool on = 64 * y + lane < nn;
                    e[y] = on ? arc_at(64 * y + lane) : 0u;
                    v[y] = on ? R.rec[e[y]] : 0ull;
                    wt[y] = kBits == 32 && on ? R.wout[e[y]] : kIc && on ? R.thr[e[y]] : 0ull;
                }
                wait_loads();
#pragma unroll
                for (uint32_t y = 0; y < kSlots; ++y) {
                    fresh[y] = false;
                    if (64 * y >= nn) continue;
                    fresh[y] = 64 * y + lane < nn && crosses(rec_node(v[y]), wt[y], e[y]);
                }
                append(fresh, v);
            };
            for (uint32_t win = 0; win < total; win += kLiveBuf) {
                const uint32_t p = incl - c - win;  // wraps below the window
                __builtin_amdgcn_wave_barrier();
                for (uint32_t k = 0; k < c; ++k)
                    if (p + k < kLiveBuf) buf[p + k] = o0 + k;
                __builtin_amdgcn_wave_barrier();
                visit_arcs([&](uint32_t k) { return buf[k]; }, total - win < kLiveBuf ? total - win : kLiveBuf);
            }
            uint64_t longs = __ballot(deg > kLaneArcs);
            while (longs) {
                const int j = __builtin_ctzll(longs);
                longs &= longs - 1;
                const uint32_t a0 = (uint32_t)__builtin_amdgcn_readlane((int)o0, j);
                const uint32_t a1 = a0 + (uint32_t)__builtin_amdgcn_readlane((int)deg, j);
                for (uint32_t k0 = a0; k0 < a1; k0 += kLiveBuf)
                    visit_arcs([&](uint32_t k) { return k0 + k; }, a1 - k0 < kLiveBuf ? a1 - k0 : kLiveBuf);
            }
        }
        if (R.bitmaps && (kLds || kBits != 32)) {
            uint32_t* out = R.bitmaps + (uint64_t)row * bm_words;
            for (uint32_t i = threadIdx.x; i < bm_words; i += 64 * kW) {
                uint32_t x = 0;
                if constexpr (kBits == 32 || kIc) {
                    x = bm[i];
                } else {
                    // the active bits of 32 nodes
#pragma unroll
                    for (uint32_t y = 0; y < 32 / kPer; ++y) {
                        const uint32_t at = i * (32 / kPer) + y;
                        const uint32_t s = at >= st_words ? 0u : kLds ? st[at] : load_relaxed32(&st[at]);
#pragma unroll
                        for (uint32_t q = 0; q < kPer; ++q)
                            x |= ((s >> (q * kBits + kBits - 1)) & (32 * i + y * kPer + q < n ? 1u : 0u)) << (y * kPer + q);
                    }
                }
                out[i] = x;
            }
        }
        if (threadIdx.x == 0) R.trial_counts[R.t0 + row] = tail;
        sum += tail;
        max_rounds = rounds > max_rounds ? rounds : max_rounds;
        __syncthreads();
    }
    if (threadIdx.x == 0 && sum) atomicAdd((unsigned long long*)R.total, (unsigned long long)sum);
    if (lane == 0 && (kIc || threadIdx.x == 0) && max_rounds > load_relaxed32(&R.status[0])) atomicMax(&R.status[0], max_rounds);
}

}  // namespace imsim
