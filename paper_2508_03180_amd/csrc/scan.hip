// Single-pass exclusive prefix sum with decoupled look-back, plus the key
// emission and tile-range kernels of cell rasterization (Sec. IV-B).  The
// primitives are first sorted by depth (ties by id); the offsets of their
// keys come from a scan over that order, so the emitted sequence is already
// in (depth, id) order within every tile and a stable sort on the tile bits
// alone completes the (tile, depth) order.
#include <string.h>

#include "common.h"
#include "launch.h"

namespace dgs {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanPart = kScanThreads * kScanItems;
constexpr int kOwnTiles = 32;

constexpr int kSpinLimit = 1 << 22;

// status word: epoch << 34 | flag << 32 | value; flag 1 = partition total,
// 2 = inclusive prefix.  Words from an older epoch read as unpublished.
__device__ inline uint64_t ld_status(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_status(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Inclusive scan across the 64 lanes of a wavefront.
__device__ inline uint32_t wave_incl_scan(uint32_t v) {
    int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

__device__ inline uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Persistent blocks take partitions from a ticket counter in launch order, so
// a partition only ever waits for partitions that are already running.
__global__ __launch_bounds__(kScanThreads) void k_scan_excl(const uint32_t* __restrict__ in,
                                                             uint32_t* __restrict__ out, int64_t n,
                                                             uint32_t* __restrict__ total, uint64_t* status,
                                                             const uint32_t* ep, uint32_t* ticket, int* err,
                                                             const uint32_t* __restrict__ idx) {
    __shared__ uint32_t s_part, s_wsum[kScanThreads / 64], s_excl;
    const uint32_t epoch = epoch_tag(*ep, 0);
    const int nparts = (int)((n + kScanPart - 1) / kScanPart);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (;;) {
        if (tid == 0) s_part = atomicAdd(ticket, 1u);
        __syncthreads();
        const int part = (int)__builtin_amdgcn_readfirstlane(s_part);  // uniform: scalar loop control
        if (part >= nparts) break;
        const int64_t base = (int64_t)part * kScanPart + (int64_t)tid * kScanItems;
        uint32_t x[kScanItems], sum = 0;
#pragma unroll
        for (int i = 0; i < kScanItems; i++) {
            uint32_t j = (uint32_t)(base + i);
            if (idx && base + i < n) j = idx[base + i];  // a permutation of [0, n)
            x[i] = (base + i < n && j < (uint64_t)n) ? in[j] : 0u;
            sum += x[i];
        }
        uint32_t incl = wave_incl_scan(sum);
        if (lane == 63) s_wsum[wave] = incl;
        __syncthreads();
        uint32_t wprefix = 0, btotal = 0;
        for (int w = 0; w < kScanThreads / 64; w++) {
            uint32_t s = s_wsum[w];
            if (w < wave) wprefix += s;
            btotal += s;
        }
        if (wave == 0) {
            // decoupled look-back by the whole wavefront: lane l reads the
            // status of partition j - l, so one round trip covers 64
            // predecessors; it stops at the nearest inclusive prefix
            const uint64_t tag = (uint64_t)epoch << 34;
            uint32_t excl = 0;
            if (part == 0) {
                if (lane == 0) st_status(&status[0], tag | (2ull << 32) | btotal);
            } else {
                if (lane == 0) st_status(&status[part], tag | (1ull << 32) | btotal);
                int j = part - 1, spins = 0;
                for (;;) {
                    const int idx = j - lane;
                    uint32_t flag = 2, val = 0;  // before partition 0: an inclusive prefix of 0
                    if (idx >= 0) {
                        const uint64_t st = ld_status(&status[idx]);
                        flag = (uint32_t)(st >> 34) == epoch ? (uint32_t)(st >> 32) & 3u : 0u;
                        val = (uint32_t)st;
                    }
                    const uint64_t notready = __ballot(flag == 0), inclusive = __ballot(flag == 2);
                    const int fn = notready ? __builtin_ctzll(notready) : 64;
                    const int li = inclusive ? __builtin_ctzll(inclusive) : 64;
                    if (li < fn) {  // every partition down to the nearest inclusive prefix is published
                        excl += wave_sum_u32(lane <= li ? val : 0u);
                        break;
                    }
                    if (fn > 0) {  // totals of the published run [0, fn): take them and move on
                        excl += wave_sum_u32(lane < fn ? val : 0u);
                        j -= fn;
                        continue;
                    }
                    if (++spins > kSpinLimit) {
                        if (lane == 0) atomicOr(err, (1 << kErrTimeout) | (1 << kErrWaitScan));
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                if (lane == 0) st_status(&status[part], tag | (2ull << 32) | (excl + btotal));
            }
            if (lane == 0) {
                s_excl = excl;
                if (part == nparts - 1) *total = excl + btotal;
            }
        }
        __syncthreads();
        uint32_t run = s_excl + wprefix + incl - sum;
#pragma unroll
        for (int i = 0; i < kScanItems; i++) {
            if (base + i < n) out[base + i] = run;
            run += x[i];
        }
        if (gridDim.x >= (unsigned)nparts) break;  // the other partitions went to other workgroups
        __syncthreads();  // s_part / s_wsum are reused by the next partition
    }
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

void launch_fill_u32(hipStream_t st, uint32_t* p, uint32_t v, size_t n) {
    if (n == 0) return;
    size_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, v, n);
}

// Readback by a kernel: a copy after the wait is a second submission and a
// second wait, 12 us on a 256 x 256 frame (127 -> 115 us) or a sort (223 -> 210).
__global__ void k_report(const int* err, const uint32_t* keys, uint32_t* dst) {
    if (threadIdx.x == 0) __hip_atomic_store(dst, (uint32_t)*err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (threadIdx.x == 1 && keys) __hip_atomic_store(dst + 1, *keys, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

void launch_report(hipStream_t st, const int* err, const uint32_t* keys, uint32_t* dst) {
    hipLaunchKernelGGL(k_report, dim3(1), dim3(64), 0, st, err, keys, dst);
}

size_t scan_status_words(int64_t n) { return (size_t)((n + kScanPart - 1) / kScanPart) + 1; }

void launch_exclusive_scan(hipStream_t st, const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total,
                           uint64_t* status, const uint32_t* epoch, uint32_t* ticket, int* err,
                           const uint32_t* idx) {
    if (n <= 0) {
        launch_fill_u32(st, total, 0u, 1);
        return;
    }
    const size_t nparts = (size_t)((n + kScanPart - 1) / kScanPart);
    const unsigned grid = (unsigned)(nparts < 1024 ? nparts : 1024);
    hipLaunchKernelGGL(k_scan_excl, dim3(grid), dim3(kScanThreads), 0, st, in, out, n, total, status,
                       epoch, ticket, err, idx);
}

__global__ void k_clear(ClearList l, FrameK f, FrameK* fdst) {
    const size_t gid = blockIdx.x * (size_t)blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    for (int b = 0; b < l.count; b++) {
        size_t i0 = 0;
        if (((uintptr_t)l.p[b] & 15) == 0) {  // 16 bytes per store
            uint4* p4 = reinterpret_cast<uint4*>(l.p[b]);
            const size_t n4 = l.n[b] / 4;
            for (size_t i = gid; i < n4; i += stride) p4[i] = make_uint4(0u, 0u, 0u, 0u);
            i0 = 4 * n4;
        }
        for (size_t i = i0 + gid; i < l.n[b]; i += stride) l.p[b][i] = 0u;
    }
    if (l.bump && gid == 0) *l.bump += 1u;
    if (fdst) {
        static_assert(sizeof(FrameK) % 4 == 0, "frame record in words");
        const uint32_t* src = reinterpret_cast<const uint32_t*>(&f);
        uint32_t* dst = reinterpret_cast<uint32_t*>(fdst);
        for (size_t i = gid; i < sizeof(FrameK) / 4; i += stride) dst[i] = src[i];
    }
}

void launch_clear(hipStream_t st, const ClearList& l, const FrameK* f, FrameK* fdst) {
    size_t most = 0;
    for (int b = 0; b < l.count; b++) most = l.n[b] > most ? l.n[b] : most;
    if (most == 0) most = 1;
    const size_t blocks = (most + 1023) / 1024;
    const unsigned grid = (unsigned)(blocks > 2048 ? 2048 : blocks);
    FrameK fv;
    if (f) fv = *f;
    else memset(&fv, 0, sizeof(fv));
    hipLaunchKernelGGL(k_clear, dim3(grid), dim3(256), 0, st, l, fv, f ? fdst : nullptr);
}

// ---------------------------------------------------------------- keys

// Depth keys of the primitives.
__global__ __launch_bounds__(256) void k_prim_keys(int P, const uint32_t* __restrict__ ntiles,
                                                   const uint32_t* __restrict__ depth, uint32_t* __restrict__ keys,
                                                   uint32_t* __restrict__ vals) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    const uint32_t d = depth[p];  // beside the count: one round trip
    keys[p] = ntiles[p] ? d : 0xffffffffu;
    vals[p] = (uint32_t)p;
}

void launch_prim_keys(hipStream_t st, int P, const uint32_t* ntiles, const uint32_t* depth, uint32_t* keys,
                      uint32_t* vals) {
    if (P <= 0) return;
    hipLaunchKernelGGL(k_prim_keys, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, st, P, ntiles, depth, keys, vals);
}

// Key emission in depth order.  A lane writes the keys of its own primitive
// up to kOwnTiles; those of a larger one are dealt over the wavefront (one
// lane writing the up to 32,400 keys of a screen-filling cell held a 4K frame
// for 2.7 ms).
__global__ __launch_bounds__(256) void k_emit_keys(int P, const uint32_t* __restrict__ order,
                                                   const uint32_t* __restrict__ ntiles,
                                                   const uint32_t* __restrict__ offsets,
                                                   const uint64_t* __restrict__ prect,
                                                   const uint32_t* __restrict__ depth, int TX, uint32_t cap,
                                                   uint64_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                   int* err) {
    const int lane = threadIdx.x & 63, i0 = blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t p = (uint32_t)P;
    if (i0 < P) p = order ? order[i0] : (uint32_t)i0;  // null order: id order
    // a permutation of [0, P) unless a scan wait timed out
    uint32_t nt = 0, off = 0, d = 0, t00 = 0, w = 0;
    if (p < (uint32_t)P) nt = ntiles[p];
    if (nt) {
        off = offsets[i0];
        if ((uint64_t)off + nt > cap) atomicOr(err, 1 << kErrCapacity);
        const uint64_t r = prect[p];
        d = depth[p];
        const int tx0 = rect_x0(r) / kTile, ty0 = rect_y0(r) / kTile;
        w = (uint32_t)(rect_x1(r) / kTile - tx0 + 1);
        t00 = (uint32_t)(ty0 * TX + tx0);
    }
    if (nt <= (uint32_t)kOwnTiles)
        for (uint32_t i = off, t0 = t00, done = 0; done < nt && i < cap; done += w, t0 += (uint32_t)TX) {
            // one row of tiles: consecutive tile ids t0 .. t0 + kept - 1
            const uint32_t kept = cap - i < w ? cap - i : w;
            for (uint32_t j = 0; j < kept; j++) {
                keys[i + j] = ((uint64_t)(t0 + j) << 32) | d;
                vals[i + j] = p;
            }
            i += kept;
        }
    for (uint64_t m = __ballot(nt > (uint32_t)kOwnTiles); m; m &= m - 1) {
        const int l = __builtin_ctzll(m);
        const uint32_t bn = (uint32_t)__builtin_amdgcn_readlane((int)nt, l), bw = (uint32_t)__builtin_amdgcn_readlane((int)w, l);
        const uint32_t bo = (uint32_t)__builtin_amdgcn_readlane((int)off, l), bt = (uint32_t)__builtin_amdgcn_readlane((int)t00, l);
        const uint32_t bd = (uint32_t)__builtin_amdgcn_readlane((int)d, l), bp = (uint32_t)__builtin_amdgcn_readlane((int)p, l);
        const uint32_t keep = bo < cap ? min(bn, cap - bo) : 0u;  // keys below the capacity
        // k / bw through a double: exact for k < 2^32 / bw with (k + 0.5) / bw
        // at least 0.5 / bw off any integer
        const double inv = 1.0 / (double)bw;
        for (uint32_t k = lane; k < keep; k += 64) {
            const uint32_t row = (uint32_t)(((double)k + 0.5) * inv);
            keys[bo + k] = ((uint64_t)(bt + row * (uint32_t)TX + (k - row * bw)) << 32) | bd;
            vals[bo + k] = bp;
        }
    }
}

void launch_emit_keys(hipStream_t st, int P, const uint32_t* order, const uint32_t* ntiles,
                      const uint32_t* offsets, const uint64_t* prect, const uint32_t* depth, int TX, uint32_t cap,
                      uint64_t* keys, uint32_t* vals, int* err) {
    if (P <= 0) return;
    hipLaunchKernelGGL(k_emit_keys, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, st, P, order, ntiles, offsets,
                       prect, depth, TX, cap, keys, vals, err);
}

__global__ __launch_bounds__(256) void k_tile_ranges(const uint64_t* __restrict__ keys,
                                                     const uint32_t* __restrict__ n_ptr, uint32_t cap,
                                                     uint32_t* __restrict__ ranges,
                                                     const uint32_t* __restrict__ vin, uint32_t* __restrict__ vout,
                                                     uint64_t* load, uint32_t tiles) {
    uint32_t n = *n_ptr;
    if (load && blockIdx.x == 0 && threadIdx.x == 0)  // the frame's load, for the host (pinned memory)
        __hip_atomic_store(load, ((uint64_t)tiles << 32) | n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (n > cap) n = cap;
    // the tile words of the neighbours (at clamped indexes) and the value
    // are loaded at once, before any of them is compared
    const uint32_t* tw = reinterpret_cast<const uint32_t*>(keys) + 1;  // tile of key i: tw[2 i]
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint32_t t = tw[2 * (size_t)i];
        const uint32_t tp = tw[2 * (size_t)(i > 0 ? i - 1 : 0)];
        const uint32_t tn = tw[2 * (size_t)(i + 1 < n ? i + 1 : i)];
        const uint32_t v = vout ? vin[i] : 0u;
        if (i == 0 || tp != t) ranges[2 * t] = i;
        if (i == n - 1 || tn != t) ranges[2 * t + 1] = i + 1;
        if (vout) vout[i] = v;
    }
}

void launch_tile_ranges(hipStream_t st, const uint64_t* keys, const uint32_t* n_ptr, uint32_t cap,
                        uint32_t* ranges, const uint32_t* vin, uint32_t* vout, uint64_t* load, uint32_t tiles) {
    unsigned grid = (unsigned)((cap + 255) / 256);
    if (grid > 2048) grid = 2048;
    if (grid == 0) grid = 1;
    hipLaunchKernelGGL(k_tile_ranges, dim3(grid), dim3(256), 0, st, keys, n_ptr, cap, ranges, vin, vout, load, tiles);
}

}  // namespace dgs
