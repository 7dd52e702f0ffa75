// The key offsets, key emission and tile-range kernels of cell rasterization
// (Sec. IV-B), and small fills and readbacks.  The
// primitives are first sorted by depth (ties by id); the offsets of their
// keys come from a scan over that order, so the emitted sequence is already
// in (depth, id) order within every tile and a stable sort on the tile bits
// alone completes the (tile, depth) order.
#include <string.h>

#include "common.h"
#include "launch.h"

namespace dgs {

// Primitives per workgroup of k_prim_offsets.
constexpr int kOffsetBlock = 1024;

// Inclusive scan across the 64 lanes of a wavefront.
__device__ inline uint32_t wave_incl_scan(uint32_t v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
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

size_t scan_status_words(int64_t n) { return (size_t)((n + 2 * kOffsetBlock - 1) / (2 * kOffsetBlock)) + 1; }

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

// Offsets of the primitives' keys in depth order, first within blocks of
// kOffsetBlock primitives with the blocks' sums, then (k_block_offsets) of the
// blocks.  One scan of the whole order whose partitions waited for each other
// took 22 us for 1 M primitives, mostly for the wait; these take 17 (with the rectangles) and 5.
// The rectangles, which the tile counts come from, are also left in depth
// order: a gather in that order moves a line for each of its words, so there is
// this one and the emission reads in sequence.
__global__ __launch_bounds__(256) void k_prim_offsets(int P, DepthOrder o, const uint64_t* __restrict__ prect,
                                                      uint32_t* __restrict__ offsets, uint32_t* __restrict__ sums) {
    constexpr int kItems = kOffsetBlock / 256;
    __shared__ uint32_t s_wsum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = blockIdx.x * kOffsetBlock + threadIdx.x * kItems;
    uint32_t p[kItems], x[kItems], sum = 0;
    uint64_t r[kItems];
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        // all ones: touches no tile (launch_prim_keys)
        const bool in = i0 + i < P && o.depth[i0 + i] != 0xffffffffu;
        p[i] = in ? o.id[i0 + i] : (uint32_t)P;
    }
#pragma unroll
    for (int i = 0; i < kItems; i++) r[i] = p[i] < (uint32_t)P ? prect[p[i]] : 0u;
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const int w = rect_x1(r[i]) / kTile - rect_x0(r[i]) / kTile + 1;
        const int h = rect_y1(r[i]) / kTile - rect_y0(r[i]) / kTile + 1;
        x[i] = p[i] < (uint32_t)P ? (uint32_t)(w * h) : 0u;
        sum += x[i];
        if (i0 + i < P) {
            o.rx[i0 + i] = (uint32_t)r[i];
            o.ry[i0 + i] = (uint32_t)(r[i] >> 32);
        }
    }
    const uint32_t incl = wave_incl_scan(sum);
    if (lane == 63) s_wsum[wave] = incl;
    __syncthreads();
    uint64_t run = incl - sum;
    for (int w = 0; w < wave; w++) run += s_wsum[w];
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        if (i0 + i < P) offsets[i0 + i] = (uint32_t)run;
        run += x[i];
    }
    if (threadIdx.x == 255) sums[blockIdx.x] = (uint32_t)min(run, (uint64_t)0xffffffffu);
}

// sums -> exclusive prefixes, in place; *total = their sum (both at most
// 2^32 - 1).  One workgroup.
__global__ __launch_bounds__(1024) void k_block_offsets(uint32_t* __restrict__ sums, uint32_t blocks, uint32_t cap,
                                                        uint32_t* __restrict__ total, int* err) {
    constexpr uint32_t kItems = 4;
    __shared__ uint64_t s_wsum[16];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint64_t carry = 0;
    for (uint32_t b0 = 0; b0 < blocks; b0 += 1024 * kItems) {
        const uint32_t b = b0 + tid * kItems;
        uint32_t x[kItems];
        uint64_t sum = 0;
#pragma unroll
        for (uint32_t i = 0; i < kItems; i++) x[i] = b + i < blocks ? sums[b + i] : 0u;
#pragma unroll
        for (uint32_t i = 0; i < kItems; i++) sum += x[i];
        uint64_t incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t u = __shfl_up(incl, d, 64);
            if (lane >= (uint32_t)d) incl += u;
        }
        if (lane == 63) s_wsum[wave] = incl;
        __syncthreads();
        uint64_t run = carry + incl - sum;
        for (uint32_t w = 0; w < 16; w++) {
            const uint64_t s = s_wsum[w];
            if (w < wave) run += s;
            carry += s;
        }
#pragma unroll
        for (uint32_t i = 0; i < kItems; i++) {
            if (b + i < blocks) sums[b + i] = (uint32_t)min(run, (uint64_t)0xffffffffu);
            run += x[i];
        }
        __syncthreads();  // s_wsum is written again
    }
    if (tid == 0) {
        *total = (uint32_t)min(carry, (uint64_t)0xffffffffu);
        if (carry > cap) atomicOr(err, 1 << kErrCapacity);
    }
}

// Key emission in depth order, a workgroup per kEmitKeys consecutive keys
// whatever their primitives' sizes: it finds the first key's primitive in the
// blocks' and the block's offsets, marks the places where the following
// primitives begin and spreads them by a maximum scan.  The stores are
// consecutive.  3.2 M keys of 1 M primitives 17 us, 35 with a lane or (beyond
// 32 tiles) a wavefront per primitive, which took 1043 us for 13.7 M keys of
// 600,000 cells, some of 32,400 tiles (the frame 1846 us, now 950).
constexpr int kEmitKeys = 2048;
// Workgroups of a grid for the capacity; beyond them each takes several blocks
// of keys (LOOP), as in the sort.
constexpr unsigned kMaxEmitGrid = 16384;
template <bool LOOP>
__global__ __launch_bounds__(256) void k_emit_keys(int P, DepthOrder order, const uint32_t* __restrict__ offsets,
                                                   const uint32_t* __restrict__ blocks,
                                                   const uint32_t* __restrict__ total, int TX, uint32_t cap,
                                                   uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
    constexpr int kItems = kEmitKeys / 256;
    __shared__ uint32_t s_off[kEmitKeys];                     // offset of primitive first + i, minus k0
    __shared__ __align__(16) uint16_t s_own[kEmitKeys];       // the key's primitive, minus first
    __shared__ uint32_t s_wave[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t n = min(*total, cap);
    uint32_t k0 = blockIdx.x * (uint32_t)kEmitKeys;
    for (; k0 < n; k0 += gridDim.x * (uint32_t)kEmitKeys) {
        const uint32_t cnt = min(n - k0, (uint32_t)kEmitKeys);
        // the number of the workgroup's 256 flags, in every thread
        const auto count = [&](bool f) {
            const uint32_t c = (uint32_t)__popcll(__ballot(f));
            if (lane == 0) s_wave[wave] = c;
            __syncthreads();
            const uint32_t r = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
            __syncthreads();  // s_wave is written again
            return r;
        };
        // the block of the first key's primitive: the last that begins at or before it
        uint32_t lo = 0, hi = (uint32_t)((P + kOffsetBlock - 1) / kOffsetBlock);
        while (hi - lo > 1) {  // blocks[lo] <= k0
            const uint32_t step = (hi - lo + 255) / 256, b = lo + tid * step;
            const uint32_t c = count(b < hi && blocks[b] <= k0);  // at least thread 0's
            lo += (c - 1) * step;
            hi = min(hi, lo + step);
        }
        const uint32_t bo = k0 - blocks[lo], q = lo * kOffsetBlock + tid * 4;
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < 4; i++)
            c += (uint32_t)__popcll(__ballot(q + i < (uint32_t)P && offsets[min(q + i, (uint32_t)P - 1)] <= bo));
        if (lane == 0) s_wave[wave] = c;
        __syncthreads();
        const uint32_t first = lo * kOffsetBlock + s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3] - 1;
        // the primitives from there on: every one before n has a key, so the
        // workgroup's keys are of at most kEmitKeys of them
#pragma unroll
        for (int i = 0; i < kItems; i++) s_own[tid + 256 * i] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kItems; i++) {
            const uint32_t l = tid + 256 * i, g = first + l;
            if (g < (uint32_t)P) {
                const uint32_t o = key_place(blocks[g / kOffsetBlock], offsets[g], k0);  // negative for the first
                s_off[l] = o;
                if (l > 0 && o < cnt) s_own[o] = (uint16_t)l;
            }
        }
        __syncthreads();
        // maximum over the keys up to each one: eight consecutive per thread
        {
            const uint4 v = reinterpret_cast<const uint4*>(s_own)[tid];
            uint32_t m[8] = {v.x & 0xffffu, v.x >> 16, v.y & 0xffffu, v.y >> 16,
                             v.z & 0xffffu, v.z >> 16, v.w & 0xffffu, v.w >> 16};
#pragma unroll
            for (int i = 1; i < 8; i++) m[i] = max(m[i], m[i - 1]);
            uint32_t x = m[7];
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t u = __shfl_up(x, d, 64);
                if (lane >= d) x = max(x, u);
            }
            if (lane == 63) s_wave[wave] = x;
            uint32_t before = __shfl_up(x, 1, 64);
            if (lane == 0) before = 0;
            __syncthreads();
            for (int w = 0; w < wave; w++) before = max(before, s_wave[w]);
            uint32_t h[4];
#pragma unroll
            for (int i = 0; i < 4; i++) h[i] = max(m[2 * i], before) | max(m[2 * i + 1], before) << 16;
            reinterpret_cast<uint4*>(s_own)[tid] = make_uint4(h[0], h[1], h[2], h[3]);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kItems; i++) {
            const uint32_t k = tid + 256 * i;
            if (k >= cnt) break;
            const uint32_t l = s_own[k], j = k - s_off[l], g = first + l;
            const uint64_t r = order.rx[g] | (uint64_t)order.ry[g] << 32;
            const int tx0 = rect_x0(r) / kTile, ty0 = rect_y0(r) / kTile;
            const uint32_t w = (uint32_t)(rect_x1(r) / kTile - tx0 + 1);
            // j / w by a reciprocal, at most one off (j < 2^24)
            uint32_t row = (uint32_t)(((float)j + 0.5f) * __builtin_amdgcn_rcpf((float)w));
            int col = (int)(j - row * w);
            if (col < 0) {
                col += (int)w;
                row--;
            } else if (col >= (int)w) {
                col -= (int)w;
                row++;
            }
            keys[k0 + k] = ((uint64_t)((ty0 + row) * (uint32_t)TX + (uint32_t)(tx0 + col)) << 32) | order.depth[g];
            vals[k0 + k] = order.id[g];
        }
        if (!LOOP) return;
        __syncthreads();  // the LDS is written again
    }
}

void launch_emit_keys(hipStream_t st, int P, const DepthOrder& order, const uint64_t* prect, uint32_t* offsets,
                      uint32_t* sums, int TX, uint32_t cap, uint64_t* keys, uint32_t* vals, uint32_t* total, int* err) {
    if (P <= 0) {
        launch_fill_u32(st, total, 0u, 1);
        return;
    }
    const unsigned blocks = (unsigned)((P + kOffsetBlock - 1) / kOffsetBlock);
    hipLaunchKernelGGL(k_prim_offsets, dim3(blocks), dim3(256), 0, st, P, order, prect, offsets, sums);
    hipLaunchKernelGGL(k_block_offsets, dim3(1), dim3(1024), 0, st, sums, blocks, cap, total, err);
    const unsigned groups = (unsigned)(((uint64_t)cap + kEmitKeys - 1) / kEmitKeys);
    if (groups > kMaxEmitGrid)
        hipLaunchKernelGGL(k_emit_keys<true>, dim3(kMaxEmitGrid), dim3(256), 0, st, P, order, offsets, sums, total, TX,
                           cap, keys, vals);
    else if (groups > 0)
        hipLaunchKernelGGL(k_emit_keys<false>, dim3(groups), dim3(256), 0, st, P, order, offsets, sums, total, TX, cap,
                           keys, vals);
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
