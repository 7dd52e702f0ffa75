// The compositor's work queue (Sec. V-B's tiles taken by persistent
// wavefronts, heaviest first), built by one workgroup of NT threads: by
// k_tile_order, or by one workgroup of the per-tile depth sort's launch.
#pragma once
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "common.h"

namespace dgs {

// Builds the work queue: per tile one whole-tile item, two half-tile items or
// four quarter-tile items, by its list's length.  Items are counting-sorted by
// estimated cost -- list length times the vector instructions a list
// entry's member costs over the item's strips -- and laid out costliest
// first, so the longest walks start at once (order within a cost class is
// arbitrary: it only affects scheduling, never results).
// queue[1] = item count, the counters are reset.  One workgroup.  With
// long_stat set (pinned host memory), also stores prims << 32 | the number
// of keys in runs of more than kLongRunKeys entries, for the host's choice
// of list order.
//
// A wavefront alone issues one instruction every four cycles, however idle
// the chip is: a half-tile item spends 58 on each member it meets (40 of them
// vector ones), a quarter (8 x 8 pixels; four members at a time) 40 (28), and
// meets fewer members, but over a tile that is 40% more vector instructions and
// twice the LDS reads.  So tiles whose list is longer than the frame's
// entries per SIMD (kSimds), which would outlast the rest of the launch, are
// cut in quarters; of the others those of at least split_len entries in
// halves.  Quarters from an eighth, a quarter, half and all of that length
// and none: the 256 x 256 frame of 2000 cells 40, 40, 40, 40, 65 us of
// compositor, 641 x 479 of 20,000 cells 180, 180, 180, 182, 269 us, but
// 1920 x 1080 of 100,000 cells 247, 237, 229, 225, 225 us.
// The items are handed out so that no counter is a bottleneck: one counter
// in memory serves about 87 tickets per us (11.4 ns each, whatever the
// workgroups), so the 4096 wavefronts of a launch took 47 us to get their
// first one, and a 4K frame's 65,000 items ran at that rate (793 us of
// compositor, 387 without it).  Here a wavefront's first item follows from its
// own number, without a ticket, and the items after those belong to kQueues
// counters (item kQueues k + q of the rest to counter q), each in a 128-byte
// line of its own; a wavefront draws from the counter of its XCD and, when
// that has run out, from the next one with items left.
//
// The list is taken from both ends: HEAVY wavefronts of a workgroup of W
// start at its costliest items and go down, the others at its cheapest and
// go up.  An item's cost is not known well (a walk ends where its pixels are
// opaque), and four costly ones on a SIMD together bind it for most of the
// launch; two, with cheap ones beside them, leave the balance to be made by
// what is taken later.  At 1920 x 1080 (100,000 cells): 4, 2 and 1 of 4
// heavy: 242, 225 and 241 us.
// The backward's items cost more and differ more: it takes them from the costly
// end only (with 2 of 4 heavy the step of 1343 us for 1285), and where there can
// be more of them than wavefronts also the first by ticket (its kernel 599 us,
// 615 with static first ones, 625 when it took the forward's list, whose quarters
// it walked as halves in the places of cheaper items; with few items tickets
// cost 5 us: 186 / 191 at 301 x 203, and 780 / 808 at 640 x 360).
constexpr int kQueues = kXcds;
constexpr int kQueueStride = 32;  // words
constexpr int kQueueWords = kQueueStride * (1 + kQueues);  // word 1: item count, line 1 + q: counter q
constexpr int kOrderClasses = 4096;
constexpr uint32_t kLongRunKeys = 4096;

struct SplitRule {
    uint32_t half, quarter;  // list lengths from which a tile is cut in 2 or 4
};

constexpr uint32_t kSimds = 1024;

// total: the frame's list entries.
__device__ __forceinline__ SplitRule split_rule(uint32_t split_len, uint32_t total) {
    return {split_len, max(split_len / 4u, total / kSimds)};
}

// The backward has a list of its own, without quarters: a Gaussian's gradient
// has a term from every item that it touches, whose order is free.
__device__ __forceinline__ SplitRule split_rule_bwd(uint32_t split_len) { return {split_len, 0xffffffffu}; }

__device__ __forceinline__ void tile_items(uint32_t len, SplitRule r, uint32_t& n, uint32_t& cls) {
    n = len >= r.quarter ? 4u : len >= r.half ? 2u : 1u;
    // Relative costs per member of a whole-tile (4 strips), a half (2 strips)
    // and a quarter walk: vector instructions of its member loop as first
    // counted.  The loops have 70, 40 and 28 now, but with those as costs a
    // ragged 1280 x 720 frame is 1.1% slower and 1920 x 1080 the same.
    const uint32_t w = n == 4u ? 29u : n == 2u ? 45u : 77u;
    const uint32_t c = (uint32_t)min((uint64_t)len * w >> 5, (uint64_t)kOrderClasses - 1u);
    cls = c;
}

// s_cnt [kOrderClasses]: counts, then the first slot of each class;
// s_part [NT / 64]: the wavefronts' sums (LDS of the calling workgroup).
template <int NT>
__device__ __forceinline__ void build_work_queue(const uint32_t* __restrict__ ranges, int ntiles, SplitRule rule,
                                        uint32_t* __restrict__ order, uint32_t* __restrict__ queue,
                                        uint32_t* s_cnt, uint32_t* s_part, int tid,
                                        uint64_t* long_stat = nullptr, uint32_t prims = 0) {
    __shared__ uint32_t s_long;
    constexpr int kAhead = 4;  // ranges loaded at once by a thread
    const uint2* rg = reinterpret_cast<const uint2*>(ranges);
    for (int i = tid; i < kOrderClasses; i += NT) s_cnt[i] = 0;
    if (tid == 0) s_long = 0;
    __syncthreads();
    uint32_t lng = 0;  // keys of this thread's tiles in runs longer than kLongRunKeys
    for (int t0 = tid; t0 < ntiles; t0 += kAhead * NT) {
        uint2 r[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; i++) r[i] = rg[min(t0 + i * NT, ntiles - 1)];
#pragma unroll
        for (int i = 0; i < kAhead; i++) {
            if (t0 + i * NT >= ntiles) break;
            uint32_t n, cls;
            const uint32_t len = r[i].y - r[i].x;
            tile_items(len, rule, n, cls);
            atomicAdd(&s_cnt[cls], n);
            lng += len > kLongRunKeys ? len : 0u;
        }
    }
    if (long_stat && lng) atomicAdd(&s_long, lng);
    __syncthreads();
    if (long_stat && tid == 0)
        __hip_atomic_store(long_stat, ((uint64_t)prims << 32) | s_long, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    // costliest first: thread i owns the classes from kOrderClasses - 1 - kPer i down
    constexpr int kPer = kOrderClasses / NT;
    uint32_t loc[kPer], run = 0;
#pragma unroll
    for (int j = 0; j < kPer; j++) {
        loc[j] = run;
        run += s_cnt[kOrderClasses - 1 - (kPer * tid + j)];
    }
    // scan of the per-thread totals: within the wavefronts, then over them
    uint32_t incl = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(incl, o, 64);
        if ((tid & 63) >= o) incl += x;
    }
    if ((tid & 63) == 63) s_part[tid >> 6] = incl;
    __syncthreads();
    uint32_t before = incl - run, items = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; w++) {
        const uint32_t x = s_part[w];
        if (w < tid >> 6) before += x;
        items += x;
    }
#pragma unroll
    for (int j = 0; j < kPer; j++) s_cnt[kOrderClasses - 1 - (kPer * tid + j)] = before + loc[j];
    if (tid == 0) queue[1] = items;
    if (tid < kQueues) *reinterpret_cast<uint64_t*>(queue + kQueueStride * (1 + tid)) = 0;
    __syncthreads();
    for (int t0 = tid; t0 < ntiles; t0 += kAhead * NT) {
        uint2 r[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; i++) r[i] = rg[min(t0 + i * NT, ntiles - 1)];
#pragma unroll
        for (int i = 0; i < kAhead; i++) {
            const int t = t0 + i * NT;
            if (t >= ntiles) break;
            uint32_t n, cls;
            tile_items(r[i].y - r[i].x, rule, n, cls);
            const uint32_t o = atomicAdd(&s_cnt[cls], n);
            // mode 0: whole tile; 2 + h: half h; 4 + q: quarter q
            if (n == 1u) order[o] = (uint32_t)t << 3;
            else for (uint32_t h = 0; h < n; h++) order[o + h] = ((uint32_t)t << 3) | (n + h);
        }
    }
}

// Where a wavefront's items come from.
struct ItemSource {
    uint32_t n, waves, heads;  // items, wavefronts, of them the heavy ones
    bool heavy;
    int q;  // the counter it draws from
};

// First item of a wavefront, of n (none: a number of at least n); H of the W
// wavefronts of a workgroup are heavy.  The workgroups that share a CU (256
// apart) put their heaviest wavefront on different SIMDs.
template <int W, int H>
__device__ __forceinline__ uint32_t first_item(int wave, uint32_t n, ItemSource& src) {
    const int slot = (wave + (int)(blockIdx.x >> 8)) & (W - 1);
    src.n = n;
    src.waves = gridDim.x * W;
    src.heads = gridDim.x * H;
    src.heavy = slot < H;
    src.q = (int)blockIdx.x & (kQueues - 1);
    const uint32_t i = (uint32_t)slot * gridDim.x + blockIdx.x;
    if (n <= src.waves || src.heavy) return i;
    return n - 1 - (i - src.heads);
}

// First item where every wavefront is heavy and items may be fewer than
// wavefronts: they fill as few workgroups as they can, but one on every CU
// before a second.  Taken from the first wavefronts of all workgroups instead, the
// 1840 halves of a 640 x 360 frame shared SIMDs while others had none (20,000
// ragged cells: backward 605 us, 461 packed; by ticket 477).
constexpr uint32_t kCus = 256;
template <int W>
__device__ __forceinline__ uint32_t first_item_packed(int wave, uint32_t n, ItemSource& src) {
    const uint32_t i = first_item<W, W>(wave, n, src);
    if (n > src.waves) return i;
    const uint32_t blocks = max((n + W - 1) / W, min(gridDim.x, kCus));
    const uint32_t slot = (uint32_t)(wave + (int)(blockIdx.x >> 8)) & (W - 1);
    return blockIdx.x < blocks ? slot * blocks + blockIdx.x : n;
}

// The wavefront's next item (n: none left).  A counter holds the items taken
// from its heavy end (low word) and from its light end (high word); both only
// grow, so every wavefront comes to an end.
__device__ __forceinline__ uint32_t next_item(uint32_t* queue, ItemSource& s, int lane) {
    if (s.n <= s.waves) return s.n;
    const uint32_t rest = s.n - s.waves;
    unsigned long long* ctr = reinterpret_cast<unsigned long long*>(queue + kQueueStride);
    constexpr int kNext = kQueueStride / 2;  // 64-bit words from counter to counter
    for (;;) {
        unsigned long long k = 0;
        if (lane == 0) k = atomicAdd(ctr + kNext * s.q, s.heavy ? 1ull : 1ull << 32);
        const uint32_t h = __builtin_amdgcn_readfirstlane((uint32_t)k), l = __builtin_amdgcn_readfirstlane((uint32_t)(k >> 32));
        const uint32_t size = (rest + kQueues - 1 - (uint32_t)s.q) / kQueues;
        if (h + l < size) return s.heads + (s.heavy ? h : size - 1 - l) * kQueues + (uint32_t)s.q;
        bool left = false;
        if (lane < kQueues) {
            const uint64_t c = __hip_atomic_load(ctr + kNext * lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            left = (uint32_t)c + (uint32_t)(c >> 32) < (rest + kQueues - 1 - (uint32_t)lane) / kQueues;
        }
        const uint32_t m = (uint32_t)__ballot(left);
        if (!m) return s.n;
        const uint32_t after = (m >> s.q) | (m << (kQueues - s.q));
        s.q = (s.q + __builtin_ctz(after)) & (kQueues - 1);
    }
}

// A wavefront's first item where none follows from its number: all are drawn
// from the counters, the costliest by whichever wavefronts come first.
__device__ __forceinline__ uint32_t first_ticket(uint32_t* queue, ItemSource& s, int lane) {
    s.waves = s.heads = 0;
    return next_item(queue, s, lane);
}

}  // namespace dgs
