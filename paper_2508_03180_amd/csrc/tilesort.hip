// Per-tile depth order (Sec. IV-B), for frames with short tile lists: each
// tile's run of entries, as the counting leaves them (bin.hip: in no order),
// is sorted by (depth bits, id) -- the (tile, depth) order with ties by id,
// as the depth sort followed by the tile sort gives it.  The (depth bits,
// id) pairs of a run are distinct, so any correct sort yields that order.
//
// Workgroups of four wavefronts, a tile each (the tiles of a workgroup lie
// far apart in the image, so that the few long runs spread over the
// workgroups).  A run of up to 256 entries is sorted by its wavefront alone,
// entry lane + 64 m in register slot m of the lane (1, 2 or 4 slots): a
// bitonic network whose exchanges between entries less than 64 apart are
// cross-lane moves (DPP and row swaps, no LDS) and the others moves between
// a lane's own slots.  The workgroup then sorts its longer runs one at a
// time with the same network spread over its wavefronts, up to 4 slots per
// lane (1024 entries), only the exchanges between wavefronts going through
// LDS (at most three of its 55 steps).  Runs longer than that are sorted in
// chunks of 1024 (of 2048 by the 16 wavefronts of k_long_sort) into a spare
// buffer and merged pairwise between that buffer and the run's own entries,
// each element's place being its index in its half plus the number of smaller
// elements in the other half (binary search).  The sorted ids go to vals, and to vcopy when set.  Every helper
// is inlined: the kernel makes no calls.
#include "common.h"
#include "launch.h"
#include "order.h"

namespace dgs {

constexpr int kTsWaves = 4;
constexpr int kTsThreads = 64 * kTsWaves;
constexpr int kTsShort = 256;            // longest run one wavefront sorts
// Longest run that a workgroup of W wavefronts sorts in registers.
constexpr int ts_chunk(int waves) { return waves == kTsWaves ? 4 * kTsThreads : 2 * 64 * waves; }
constexpr int kTsChunk = ts_chunk(kTsWaves);
// Workgroups that sort the listed longer runs, one run at a time: among the
// others' four tiles, two such runs in one workgroup were the kernel's span
// (1920 x 1080, 333,333 cells of 3 with a few runs of 3,600: frame 568 -> 503
// us).  With runs from 1,024 on listed, and 256 workgroups, views with a
// thousand of them waited here (large scene 685 -> 860 us, now 669).
constexpr unsigned kTsLongGroups = 1024;
// Frames with many keys in long runs (the per-tile order chosen by the caller) sort
// the listed ones in a launch of their own, by workgroups of 16 wavefronts, in
// about half the span a run has here: 2,000,000 single Gaussians as cells at 1920 x
// 1080, 10.9 M keys, frame 2543 -> 1622 us; 6,000,000 cells at 320 x 180, 2.3 M
// keys, 8918 -> 3603.  Where long runs are few the launch costs more than it gives.
constexpr int kLongWaves = 16;

__device__ __forceinline__ void put_sorted(uint32_t* vr, uint32_t* vcopy, int i, uint64_t v) {
    vr[i] = (uint32_t)v;
    if (vcopy) vcopy[i] = (uint32_t)v;
}

// The value that lane ^ J holds, for J a power of two below 64, without
// LDS: DPP moves for partners inside a row of 16 lanes, gfx950's row swaps
// for 16 and 32 (each returns the two operands after swapping the odd rows
// of the first with the even rows of the second, resp. the upper half of
// the first with the lower half of the second).
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane) {
    if constexpr (J == 1) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
    } else if constexpr (J == 2) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
    } else if constexpr (J == 4) {
        const int m = __builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);  // row_half_mirror: lane ^ 7
        return (uint32_t)__builtin_amdgcn_mov_dpp(m, 0x1B, 0xF, 0xF, false);     // quad_perm [3,2,1,0]: ^ 3
    } else if constexpr (J == 8) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, false);  // row_ror:8
    } else if constexpr (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (lane & 16) ? r[0] : r[1];
    } else {
        static_assert(J == 32, "lane distance");
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (lane & 32) ? r[0] : r[1];
    }
}

template <int J>
__device__ __forceinline__ uint64_t lane_xor64(uint64_t v, int lane) {
    const uint32_t lo = lane_xor<J>((uint32_t)v, lane), hi = lane_xor<J>((uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// j is a constant once the networks' loops are unrolled
__device__ __forceinline__ uint64_t lane_xor64(uint64_t v, int j, int lane) {
    switch (j) {
        case 1: return lane_xor64<1>(v, lane);
        case 2: return lane_xor64<2>(v, lane);
        case 4: return lane_xor64<4>(v, lane);
        case 8: return lane_xor64<8>(v, lane);
        case 16: return lane_xor64<16>(v, lane);
        default: return lane_xor64<32>(v, lane);
    }
}

// One bitonic compare-exchange of entry e (value v) with entry e ^ j, whose
// value is o: the lower entry of the pair keeps the smaller value in an
// ascending block, the larger in a descending one.  ej: bit j of e is set
// (the upper entry); ek: bit k of e is set (a descending block of the k-merge).
__device__ __forceinline__ uint64_t cx(uint64_t v, uint64_t o, bool ej, bool ek) {
    return ((v < o) == (ej == ek)) ? v : o;
}

// Bits 0..5 of the lane index (each a lane mask the compiler can keep in
// scalar registers).
struct LaneBits {
    bool b[6];
    __device__ __forceinline__ explicit LaneBits(int lane) {
#pragma unroll
        for (int i = 0; i < 6; i++) b[i] = (lane >> i) & 1;
    }
    __device__ __forceinline__ bool operator[](int pow2) const { return b[__builtin_ctz(pow2)]; }
};

// The stages of a bitonic network over P entries held by consecutive
// wavefronts, entry base + lane + 64 m in v[m] of wavefront base / (64 M)
// (base a multiple of 64 M), that stay inside the wavefront: exchanges
// 64 or more apart between a lane's slots, shorter ones across lanes.
// Stages j >= 64 M need another wavefront's entries: xchg(k, j) does those.
template <int M, class Xchg>
__device__ __forceinline__ void bitonic(uint64_t (&v)[M], int P, int base, int lane, Xchg xchg) {
    const LaneBits lb(lane);
#pragma unroll
    for (int k = 2; k <= P; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j >= 64 * M) {
                xchg(k, j);
            } else if (j >= 64) {  // slots m and m ^ (j / 64) of the lane
#pragma unroll
                for (int m = 0; m < M; m++) {
                    const int pm = m ^ (j >> 6);
                    if (pm > m) {
                        const bool up = ((base + 64 * m) & k) == 0;
                        const uint64_t x = v[m], y = v[pm];
                        const bool sw = (x > y) == up;
                        v[m] = sw ? y : x;
                        v[pm] = sw ? x : y;
                    }
                }
            } else {
#pragma unroll
                for (int m = 0; m < M; m++) {
                    const bool ek = k < 64 ? lb[k] : ((base + 64 * m) & k) != 0;
                    v[m] = cx(v[m], lane_xor64(v[m], j, lane), lb[j], ek);
                }
            }
        }
    }
}

// A run of at most P <= 64 M entries sorted by one wavefront (the padding
// holds the largest value); with M = 1 and P < 64 the network stops at
// blocks of P lanes.
template <int M, int P = 64 * M>
__device__ __forceinline__ void wave_sort_run(const uint64_t* __restrict__ kr, uint32_t* __restrict__ vr,
                                              uint32_t* vc, int L, int lane) {
    uint64_t v[M];
#pragma unroll
    for (int m = 0; m < M; m++) {
        const int e = lane + 64 * m;
        v[m] = e < L ? kr[e] : ~0ull;  // (depth bits, id)
    }
    bitonic<M>(v, P, 0, lane, [](int, int) {});
#pragma unroll
    for (int m = 0; m < M; m++) {
        const int e = lane + 64 * m;
        if (e < L) put_sorted(vr, vc, e, v[m]);
    }
}

// A run of at most 64 W M entries sorted by W wavefronts of the workgroup
// (tid: the thread's index among them): wavefront w holds entries
// w 64 M + lane + 64 m (the padding holds the largest value); the stages
// between wavefronts go through LDS (sd, 64 W M entries).  With out set the
// sorted entries [0, L) go there instead of back into the run.
// Its barriers are the workgroup's: every wavefront of the workgroup runs
// the same network at the same time.
template <int M, int W = kTsWaves>
__device__ __forceinline__ void group_sort_run(uint64_t* sd, const uint64_t* __restrict__ kr, uint32_t* __restrict__ vr,
                                               uint32_t* vc, uint64_t* out, int L, int tid) {
    constexpr int B = 64 * M;
    const int w = tid >> 6, lane = tid & 63, base = w * B;
    uint64_t v[M];
#pragma unroll
    for (int m = 0; m < M; m++) {
        const int e = base + lane + 64 * m;
        v[m] = e < L ? kr[e] : ~0ull;  // (depth bits, id)
    }
    bitonic<M>(v, 64 * W * M, base, lane, [&](int k, int j) {
#pragma unroll
        for (int m = 0; m < M; m++) sd[base + lane + 64 * m] = v[m];
        __syncthreads();
#pragma unroll
        for (int m = 0; m < M; m++) {
            const int e = base + lane + 64 * m;
            v[m] = cx(v[m], sd[e ^ j], (e & j) != 0, (e & k) != 0);
        }
        __syncthreads();
    });
#pragma unroll
    for (int m = 0; m < M; m++) {
        const int e = base + lane + 64 * m;
        if (e < L) {
            if (out) out[e] = v[m];
            else put_sorted(vr, vc, e, v[m]);
        }
    }
}

// By a whole workgroup of W wavefronts, up to ts_chunk(W) entries.
template <int W>
__device__ __forceinline__ void group_sort_any(uint64_t* sd, const uint64_t* kr, uint32_t* vr, uint32_t* vc, uint64_t* out,
                                               int L, int tid) {
    constexpr int M = ts_chunk(W) / (64 * W);
    if (L <= ts_chunk(W) / 2) group_sort_run<M / 2, W>(sd, kr, vr, vc, out, L, tid);
    else group_sort_run<M, W>(sd, kr, vr, vc, out, L, tid);
}

// Number of entries of the ascending array y[0, n) below v.
__device__ __forceinline__ int count_below(const uint64_t* y, int n, uint64_t v) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if (y[m] < v) lo = m + 1;
        else hi = m;
    }
    return lo;
}

// One run of more than kTsShort entries, by the whole workgroup of W wavefronts
// (sd: its LDS, ts_chunk(W) entries).
template <int W>
__device__ __forceinline__ void sort_long_run(uint64_t* sd, uint32_t s, int L,
                                              uint64_t* __restrict__ ent, uint32_t* __restrict__ vals,
                                              uint64_t* __restrict__ spare, uint32_t* __restrict__ vcopy, int tid) {
    constexpr int kChunk = ts_chunk(W), kThreads = 64 * W;
    uint64_t* kr = ent + s;
    uint32_t* vr = vals + s;
    uint32_t* vc = vcopy ? vcopy + s : nullptr;
    // A run of up to kChunk entries is one chunk sorted straight back into
    // place; a longer one is sorted in chunks into the spare buffer, then
    // merged pairwise.  (One call site: the network is inlined once.)
    const bool chunked = L > kChunk;
    uint64_t* a = spare + s;
    for (int c0 = 0; c0 < L; c0 += kChunk) {
        group_sort_any<W>(sd, kr + c0, vr + c0, vc, chunked ? a + c0 : nullptr, min(kChunk, L - c0), tid);
        __syncthreads();  // sd is reused by the next chunk
    }
    if (!chunked) return;
    __threadfence_block();
    __syncthreads();
    uint64_t* src = a;
    uint64_t* dst = kr;  // the run's own entries (every one has been read)
    for (int w = kChunk; w < L; w <<= 1) {
        for (int i = tid; i < L; i += kThreads) {
            const int x0 = (i / (2 * w)) * (2 * w), y0 = x0 + w;
            const uint64_t v = src[i];
            if (i < y0) {  // in the first run of the pair
                const int yn = y0 < L ? min(w, L - y0) : 0;
                dst[i + count_below(src + y0, yn, v)] = v;
            } else {
                dst[x0 + (i - y0) + count_below(src + x0, w, v)] = v;
            }
        }
        __threadfence_block();
        __syncthreads();
        uint64_t* t = src;
        src = dst;
        dst = t;
    }
    for (int i = tid; i < L; i += kThreads) put_sorted(vr, vc, i, src[i]);
}

// The listed runs, one at a time by a workgroup of W wavefronts, number `first`
// of `groups`.
template <int W>
__device__ __forceinline__ void sort_listed_runs(uint64_t* sd, const uint32_t* __restrict__ ranges,
                                                 const uint32_t* __restrict__ long_tiles, uint32_t n, uint32_t first,
                                                 uint32_t groups, uint64_t* __restrict__ ent, uint32_t* __restrict__ vals,
                                                 uint64_t* __restrict__ spare, uint32_t* __restrict__ vcopy, int tid) {
#pragma unroll 1
    for (uint32_t i = first; i < n; i += groups) {
        const uint32_t t = long_tiles[i], s = ranges[2 * t];
        sort_long_run<W>(sd, (uint32_t)__builtin_amdgcn_readfirstlane(s),
                         __builtin_amdgcn_readfirstlane((int)(ranges[2 * t + 1] - s)), ent, vals, spare, vcopy, tid);
        __syncthreads();  // sd is reused by the next run
    }
}

__global__ __launch_bounds__(64 * kLongWaves) __attribute__((amdgpu_waves_per_eu(8))) void k_long_sort(
    const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ long_tiles, const uint32_t* __restrict__ nlong,
    uint64_t* __restrict__ ent, uint32_t* __restrict__ vals, uint64_t* __restrict__ spare, uint32_t* __restrict__ vcopy) {
    __shared__ uint64_t sd[ts_chunk(kLongWaves)];
    sort_listed_runs<kLongWaves>(sd, ranges, long_tiles, *nlong, blockIdx.x, gridDim.x, ent, vals, spare, vcopy,
                                 (int)threadIdx.x);
}

// A workgroup's LDS: the work queue's counts and partial sums (order.h), or
// the sort's exchange buffer.
constexpr int kQueueBytes = (kOrderClasses + kTsThreads) * 4;
constexpr int kTsSharedBytes = kQueueBytes > kTsChunk * 8 ? kQueueBytes : kTsChunk * 8;

// Workgroup 0 builds the compositor's work queue (it needs the tile ranges
// only), for a saved frame workgroup 1 its backward's; the others sort the runs.
__global__ __launch_bounds__(kTsThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_tile_sort(
    const uint32_t* __restrict__ ranges, int tiles, const uint32_t* __restrict__ long_tiles,
    const uint32_t* __restrict__ nlong, int long_groups, uint64_t* __restrict__ ent, uint32_t* __restrict__ vals,
    uint64_t* __restrict__ spare, uint32_t* __restrict__ vcopy, uint32_t split_len, const uint32_t* __restrict__ total,
    WorkQueue fwd, WorkQueue bwd, uint64_t* long_stat, uint32_t prims) {
    __shared__ __align__(16) unsigned char smem[kTsSharedBytes];
    __shared__ int lt_s[kTsWaves], lt_len[kTsWaves];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int queues = bwd.queue ? 2 : 1;
    if ((int)blockIdx.x < queues) {
        uint32_t* s_cnt = reinterpret_cast<uint32_t*>(smem);
        const bool b = blockIdx.x == 1;
        build_work_queue<kTsThreads>(ranges, tiles, b ? split_rule_bwd(split_len) : split_rule(split_len, *total),
                                     b ? bwd.order : fwd.order, b ? bwd.queue : fwd.queue, s_cnt,
                                     s_cnt + kOrderClasses, tid, b ? nullptr : long_stat, prims);
        return;
    }
    const int block = (int)blockIdx.x - queues;
    uint64_t* sd = reinterpret_cast<uint64_t*>(smem);
    if (block < long_groups) {
        sort_listed_runs<kTsWaves>(sd, ranges, long_tiles, *nlong, (uint32_t)block, (uint32_t)long_groups, ent, vals, spare,
                                   vcopy, tid);
        return;
    }
    const int G = (int)gridDim.x - queues - long_groups, sb = block - long_groups;
    // wavefront w takes a tile of the w-th band of G tiles, at an offset
    // that moves by a fixed stride from band to band
    const int t = w * G + (int)(((int64_t)sb + (int64_t)w * (G * 5 / 8 + 1)) % G);
    uint32_t s = 0;
    int L = 0;
    if (t < tiles) {
        s = ranges[2 * t];
        L = (int)(ranges[2 * t + 1] - s);
    }
    if (lane == 0) {
        lt_s[w] = (int)s;
        lt_len[w] = L;
    }
    if (L > 0 && L <= kTsShort) {
        const uint64_t* kr = ent + s;
        uint32_t* vr = vals + s;
        uint32_t* vc = vcopy ? vcopy + s : nullptr;
        if (L <= 16) wave_sort_run<1, 16>(kr, vr, vc, L, lane);
        else if (L <= 32) wave_sort_run<1, 32>(kr, vr, vc, L, lane);
        else if (L <= 64) wave_sort_run<1>(kr, vr, vc, L, lane);
        else if (L <= 128) wave_sort_run<2>(kr, vr, vc, L, lane);
        else wave_sort_run<4>(kr, vr, vc, L, lane);
    }
    __syncthreads();
    // the runs longer than a wavefront sorts, one at a time with the whole
    // workgroup (those beyond kLongRun are the listed ones)
#pragma unroll 1
    for (int i = 0; i < kTsWaves; i++) {
        const int len = __builtin_amdgcn_readfirstlane(lt_len[i]);
        if (len <= kTsShort || len > (int)kLongRun) continue;
        sort_long_run<kTsWaves>(sd, (uint32_t)__builtin_amdgcn_readfirstlane(lt_s[i]), len, ent, vals, spare, vcopy, tid);
        __syncthreads();  // sd is reused by the next run
    }
}

void launch_tile_depth_sort(hipStream_t st, const uint32_t* ranges, int tiles, const uint32_t* long_tiles,
                            const uint32_t* nlong, bool many_long, uint64_t* ent, uint32_t* vals, uint64_t* spare,
                            uint32_t* vcopy, uint32_t split_len, const uint32_t* total, const WorkQueue& fwd,
                            const WorkQueue& bwd, uint64_t* long_stat, uint32_t prims) {
    if (tiles <= 0) return;
    unsigned lg = (unsigned)tiles < kTsLongGroups ? (unsigned)tiles : kTsLongGroups;
    if (many_long) {
        hipLaunchKernelGGL(k_long_sort, dim3(lg), dim3(64 * kLongWaves), 0, st, ranges, long_tiles, nlong, ent, vals, spare,
                           vcopy);
        lg = 0;
    }
    // + the work queues', the long runs'
    const unsigned grid = (unsigned)((tiles + kTsWaves - 1) / kTsWaves) + (bwd.queue ? 2 : 1) + lg;
    hipLaunchKernelGGL(k_tile_sort, dim3(grid), dim3(kTsThreads), 0, st, ranges, tiles, long_tiles, nlong, (int)lg, ent, vals, spare, vcopy,
                       split_len, total, fwd, bwd, long_stat, prims);
}

__global__ __launch_bounds__(256) void k_list_keys(const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ vals,
                                                   const uint32_t* __restrict__ depth, uint64_t* __restrict__ keys) {
    const uint32_t t = blockIdx.x, end = ranges[2 * t + 1];
    for (uint32_t i = ranges[2 * t] + threadIdx.x; i < end; i += 256) keys[i] = ((uint64_t)t << 32) | depth[vals[i]];
}

void launch_list_keys(hipStream_t st, const uint32_t* ranges, int tiles, const uint32_t* vals, const uint32_t* depth,
                      uint64_t* keys) {
    if (tiles <= 0) return;
    hipLaunchKernelGGL(k_list_keys, dim3((unsigned)tiles), dim3(256), 0, st, ranges, vals, depth, keys);
}

}  // namespace dgs
