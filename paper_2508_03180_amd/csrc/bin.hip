// Tile lists by counting (Sec. IV-B), for the per-tile depth order: every
// (primitive, touched tile) entry goes straight to its tile's run, whatever
// the order inside the run, and the per-tile sort then orders each run by
// (depth bits, id).  No key is ever sorted on its tile bits:
//   k_bin_count    how many entries each chunk of primitives gives each tile
//                  (counted in LDS, one counter per tile);
//   k_bin_scan     exclusive sums of those counts over the chunks and the
//                  tiles: the first slot of every (chunk, tile), the tile
//                  ranges, the entry total;
//   k_bin_scatter  the same walk as the count, each entry taking the next
//                  slot of its (chunk, tile) from the LDS counter.
//
// The tile rows are dealt to eight bands (row ty to band ty % 8), one per
// XCD: workgroup b works on band b % 8, which is also the XCD that takes
// workgroup b, so a tile's run is written through one L2 and its 64-byte
// lines fill there before they leave (only speed depends on that placement).
// Every band's workgroups read all primitives' rectangles (8 bytes each, an
// eighth of the counters each): the counters of a 4K frame's band take 16 KB
// of LDS, and screen-filling primitives are shared by eight workgroups.
//
// Bound by latency: a few dependent trips to memory per kernel.  On the
// clustered 1M-Gaussian frame at 1920x1080 (100k cells, 0.52M entries) the
// three take 7 + 5 + 6 us by themselves, where the scan of the tile counts,
// the key emission, two radix passes on the tile bits and the tile ranges
// took 7 + 20 + 60 + 6 us; the frame went from 381 to 346 us.  Workgroups of
// 256 threads, so that they find room beside the member projection's (with
// 1024 the frame takes 358 us).
#include <algorithm>

#include "common.h"
#include "launch.h"

namespace dgs {

constexpr int kBinBands = kXcds;
constexpr int kBinThreads = 256;
constexpr int kBinPerChunk = 256;  // primitives per chunk, until there are kBinMaxChunks chunks
constexpr int kBinMaxChunks = 64;
constexpr int kBinMaxLocal = 16384;  // tiles of a band: 64 KB of LDS counters
// A lane walks the tiles of its own primitive up to this many; the tiles of
// a larger one are dealt over the wavefront's lanes.
constexpr int kBinOwnTiles = 16;
constexpr int kBinAhead = 4;  // rounds of a chunk loaded at once: 62 -> 49 us for the count of 600k cells at 4K
constexpr int kBinScanTiles = 64;                                // tiles per workgroup of the scan
constexpr int kBinScanSplit = 4;                                 // threads per tile
constexpr int kBinScanEach = kBinMaxChunks / kBinScanSplit;      // chunks per thread
constexpr int kBinSpinLimit = 1 << 22;

static int band_rows(int TY) { return (TY + kBinBands - 1) / kBinBands; }

// With c chunks the counting takes about 2.1 ns x P / c longer than with many,
// the global way 32 us + 0.05 ns x P: it is the faster one beyond
// P (kFewChunks - c) = kFewChunks kFewChunkPrims c, and never from kFewChunks on.
// Mostly culled cells at 3840 x 2160 in a tight key buffer, per tile / global
// us: 100,000 in 8, 4 and 1 chunks 291 / 313, 318 / 308 and 481 / 307; 300,000 in
// 32, 16 and 1 293 / 312, 311 / 310 and 916 / 310; 1 M in 32 and 16 358 / 376 and
// 427 / 376; 3 M in 64 and 32 456 / 537 and 549 / 531.
constexpr int64_t kFewChunks = 42, kFewChunkPrims = 15000;

// Chunks of primitives: one per kBinPerChunk of them up to kBinMaxChunks, and
// no more than `words` counters hold; 0: this grid, or these primitives with
// so few counters, take the radix sort.
int bin_chunks(int64_t P, int TX, int TY, int64_t words, size_t status_words) {
    const int64_t tiles = (int64_t)TX * TY, local = (int64_t)TX * band_rows(TY);
    if (P <= 0 || local > kBinMaxLocal || (size_t)((tiles + kBinScanTiles - 1) / kBinScanTiles) > status_words) return 0;
    const int64_t most = std::min<int64_t>((P + kBinPerChunk - 1) / kBinPerChunk, kBinMaxChunks);
    const int64_t c = std::min(most, words / (kBinBands * local));
    return P * (kFewChunks - c) > kFewChunks * kFewChunkPrims * c ? 0 : (int)c;
}

// Calls f(slot, payload) for every tile of the band that each lane's
// rectangle touches; slot = the tile's place in the band.  All lanes of the
// wavefront call it (has = false: no rectangle).
template <class F>
__device__ __forceinline__ void band_tiles(bool has, uint64_t r, uint32_t depth, uint32_t id, int band, int TX, int lane,
                                           F f) {
    int n = 0, w = 0, l0 = 0;
    if (has) {
        const int tx0 = rect_x0(r) / kTile, ty0 = rect_y0(r) / kTile, ty1 = rect_y1(r) / kTile;
        const int row = ty0 + ((band - ty0) & (kBinBands - 1));  // first row of the band
        w = rect_x1(r) / kTile - tx0 + 1;
        n = row <= ty1 ? ((ty1 - row) / kBinBands + 1) * w : 0;
        l0 = row / kBinBands * TX + tx0;
    }
    const bool big = n > kBinOwnTiles;
    if (!big)
        for (int k = 0, x = 0, s = l0; k < n; k++) {
            f(s + x, depth, id);
            if (++x == w) {
                x = 0;
                s += TX;
            }
        }
    for (uint64_t m = __ballot(big); m; m &= m - 1) {
        const int i = __builtin_ctzll(m);
        const int bn = __builtin_amdgcn_readlane(n, i), bw = __builtin_amdgcn_readlane(w, i);
        const int bl = __builtin_amdgcn_readlane(l0, i);
        const uint32_t bd = (uint32_t)__builtin_amdgcn_readlane((int)depth, i);
        const uint32_t bi = (uint32_t)__builtin_amdgcn_readlane((int)id, i);
        // k / bw through a float: (k + 0.5) / bw is at least 0.5 / bw off any
        // integer, the rounding less than 2e-7 k / bw (k < 2^14)
        const float inv = 1.0f / (float)bw;
        for (int k = lane; k < bn; k += 64) {
            const int row = (int)(((float)k + 0.5f) * inv);
            f(bl + row * TX + (k - row * bw), bd, bi);
        }
    }
}

// band_tiles over the primitives [p0, p1) of a chunk by the workgroup; the
// rectangles and depths of kBinAhead rounds are loaded at once.  A culled
// primitive's rectangle is kEmptyRect.
template <bool DEPTH, class F>
__device__ __forceinline__ void chunk_tiles(const uint64_t* __restrict__ prect, const uint32_t* __restrict__ depth, int p0,
                                            int p1, int band, int TX, int tid, F f) {
    for (int q = p0 + tid; q - tid < p1; q += kBinAhead * kBinThreads) {
        uint64_t r[kBinAhead];
        uint32_t d[kBinAhead];
#pragma unroll
        for (int i = 0; i < kBinAhead; i++) {
            const int p = q + i * kBinThreads;
            r[i] = p < p1 ? prect[p] : kEmptyRect;
            d[i] = DEPTH && p < p1 ? depth[p] : 0u;
        }
#pragma unroll
        for (int i = 0; i < kBinAhead; i++)
            band_tiles(r[i] != kEmptyRect, r[i], d[i], (uint32_t)(q + i * kBinThreads), band, TX, tid & 63, f);
    }
}

__global__ __launch_bounds__(kBinThreads) void k_bin_count(const uint64_t* __restrict__ prect, int P, int per, int TX,
                                                           int local, uint32_t* __restrict__ counts) {
    extern __shared__ uint32_t s_cnt[];
    const int tid = threadIdx.x;
    const int band = blockIdx.x & (kBinBands - 1), chunk = blockIdx.x / kBinBands;
    for (int i = tid; i < local; i += kBinThreads) s_cnt[i] = 0u;
    __syncthreads();
    chunk_tiles<false>(prect, nullptr, chunk * per, min(P, (chunk + 1) * per), band, TX, tid,
                       [&](int s, uint32_t, uint32_t) { atomicAdd(&s_cnt[s], 1u); });
    __syncthreads();
    uint32_t* out = counts + (size_t)blockIdx.x * local;
    for (int i = tid; i < local; i += kBinThreads) out[i] = s_cnt[i];
}

__global__ __launch_bounds__(kBinThreads) void k_bin_scatter(const uint64_t* __restrict__ prect,
                                                             const uint32_t* __restrict__ depth, int P, int per, int TX,
                                                             int local, const uint32_t* __restrict__ offsets, uint32_t cap,
                                                             uint64_t* __restrict__ ent) {
    extern __shared__ uint32_t s_cnt[];
    const int tid = threadIdx.x;
    const int band = blockIdx.x & (kBinBands - 1), chunk = blockIdx.x / kBinBands;
    const uint32_t* in = offsets + (size_t)blockIdx.x * local;
    for (int i = tid; i < local; i += kBinThreads) s_cnt[i] = in[i];
    __syncthreads();
    chunk_tiles<true>(prect, depth, chunk * per, min(P, (chunk + 1) * per), band, TX, tid,
                      [&](int s, uint32_t d, uint32_t id) {
                          const uint32_t pos = atomicAdd(&s_cnt[s], 1u);
                          if (pos < cap) ent[pos] = ((uint64_t)d << 32) | id;
                      });
}

// Sums saturate at 2^32 - 1, far above the largest key capacity: an overflow
// is reported and no slot beyond the capacity is written or read.  The slots
// that the scatter counts on from stop at kNoSlot instead: with the entries of
// a chunk in one tile, fewer than 2^31, they stay below 2^32.
constexpr uint32_t kNoSlot = 1u << 31;

// status word: epoch << 34 | flag << 32 | value; flag 1 = workgroup total,
// 2 = inclusive prefix.
__global__ __launch_bounds__(kBinScanTiles * kBinScanSplit) void k_bin_scan(
    uint32_t* __restrict__ counts, int chunks, int TX, int tiles, int local, uint32_t cap, uint32_t* __restrict__ ranges,
    uint32_t* __restrict__ total, uint64_t* status, const uint32_t* ep, uint32_t* ticket, uint32_t* __restrict__ long_tiles,
    uint32_t* nlong, int* err, uint64_t* load) {
    __shared__ uint32_t s_sum[kBinScanSplit][kBinScanTiles];
    __shared__ uint32_t s_wsum[kBinScanTiles / 64], s_part, s_excl;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tt = tid & (kBinScanTiles - 1), grp = tid / kBinScanTiles;
    const uint32_t epoch = epoch_tag(*ep, 0);
    if (tid == 0) s_part = atomicAdd(ticket, 1u);
    __syncthreads();
    const int part = (int)__builtin_amdgcn_readfirstlane(s_part), nparts = (int)gridDim.x;
    const int t = part * kBinScanTiles + tt;
    const int ty = t / TX, tx = t - ty * TX;
    // the counts of (chunk, tile): this thread's chunks, all loads at once
    uint32_t* col = counts + (size_t)(ty & (kBinBands - 1)) * local + (ty / kBinBands) * TX + tx;
    const size_t stride = (size_t)kBinBands * local;
    uint32_t x[kBinScanEach], sum = 0;
#pragma unroll
    for (int i = 0; i < kBinScanEach; i++) {
        const int c = grp * kBinScanEach + i;
        x[i] = t < tiles && c < chunks ? col[c * stride] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kBinScanEach; i++) sum = sat_add(sum, x[i]);
    s_sum[grp][tt] = sum;
    __syncthreads();
    uint32_t n = 0, before = 0;  // the tile's entries, and those of this thread's earlier chunks
#pragma unroll
    for (int g = 0; g < kBinScanSplit; g++) {
        if (g == grp) before = n;
        n = sat_add(n, s_sum[g][tt]);
    }
    uint32_t incl = n;  // over the wavefront's tiles (each group of threads repeats it)
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = __shfl_up(incl, d, 64);
        if (lane >= d) incl = sat_add(incl, u);
    }
    if (grp == 0 && lane == 63) s_wsum[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        uint32_t btotal = 0;
        for (int w = 0; w < kBinScanTiles / 64; w++) btotal = sat_add(btotal, s_wsum[w]);
        const uint64_t tag = (uint64_t)epoch << 34;
        uint32_t excl = 0;
        if (part > 0) {
            if (lane == 0)
                __hip_atomic_store(&status[part], tag | (1ull << 32) | btotal, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // lane l reads the word of workgroup j - l; stop at the nearest inclusive prefix
            int j = part - 1, spins = 0;
            for (;;) {
                const int idx = j - lane;
                uint32_t flag = 2, val = 0;  // before workgroup 0: an inclusive prefix of 0
                if (idx >= 0) {
                    const uint64_t st = __hip_atomic_load(&status[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    flag = (uint32_t)(st >> 34) == epoch ? (uint32_t)(st >> 32) & 3u : 0u;
                    val = (uint32_t)st;
                }
                const uint64_t notready = __ballot(flag == 0), inclusive = __ballot(flag == 2);
                const int fn = notready ? __builtin_ctzll(notready) : 64;
                const int li = inclusive ? __builtin_ctzll(inclusive) : 64;
                const bool whole = li < fn;
                uint32_t v = lane < fn && lane <= li ? val : 0u;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) v = sat_add(v, __shfl_xor(v, o, 64));
                excl = sat_add(excl, v);
                if (whole) break;
                j -= fn;
                if (fn == 0) {
                    if (++spins > kBinSpinLimit) {
                        if (lane == 0) atomicOr(err, (1 << kErrTimeout) | (1 << kErrWaitScan));
                        // unknown: everything from here on lies beyond the capacity (too
                        // small a prefix would let runs overlap, and list more long ones
                        // than long_tiles holds)
                        excl = 0xffffffffu;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
        }
        const uint32_t end = sat_add(excl, btotal);
        if (lane == 0) {
            __hip_atomic_store(&status[part], tag | (2ull << 32) | end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_excl = excl;
            if (part == nparts - 1) {
                *total = end;
                if (end > cap) atomicOr(err, 1 << kErrCapacity);
                if (load)  // the frame's load, for the host (pinned memory)
                    __hip_atomic_store(load, ((uint64_t)(uint32_t)tiles << 32) | end, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
    }
    __syncthreads();
    uint32_t start = s_excl;
    for (int w = 0; w < (wave & (kBinScanTiles / 64 - 1)); w++) start = sat_add(start, s_wsum[w]);
    const uint32_t up = __shfl_up(incl, 1, 64);
    if (lane > 0) start = sat_add(start, up);
    if (t >= tiles) return;
    if (grp == 0) {  // tiles without entries keep [0, 0)
        const uint2 r = n && start < cap ? make_uint2(start, min(sat_add(start, n), cap)) : make_uint2(0u, 0u);
        *reinterpret_cast<uint2*>(ranges + 2 * (size_t)t) = r;
        if (r.y - r.x > kLongRun) long_tiles[atomicAdd(nlong, 1u)] = (uint32_t)t;
    }
    uint32_t run = sat_add(start, before);
#pragma unroll
    for (int i = 0; i < kBinScanEach; i++) {
        const int c = grp * kBinScanEach + i;
        if (c < chunks) col[c * stride] = min(run, kNoSlot);
        run = sat_add(run, x[i]);
    }
}

void launch_bin_tiles(hipStream_t st, const BinArgs& a) {
    const int tiles = a.TX * a.TY, local = a.TX * band_rows(a.TY), chunks = a.chunks;
    const int per = (a.P + chunks - 1) / chunks;
    const dim3 grid((unsigned)(kBinBands * chunks));
    const size_t lds = (size_t)local * sizeof(uint32_t);
    hipLaunchKernelGGL(k_bin_count, grid, dim3(kBinThreads), lds, st, a.prect, a.P, per, a.TX, local, a.counts);
    hipLaunchKernelGGL(k_bin_scan, dim3((unsigned)((tiles + kBinScanTiles - 1) / kBinScanTiles)),
                       dim3(kBinScanTiles * kBinScanSplit), 0, st, a.counts, chunks, a.TX, tiles, local, a.cap, a.ranges,
                       a.total, a.status, a.epoch, a.ticket, a.long_tiles, a.nlong, a.err, a.load);
    hipLaunchKernelGGL(k_bin_scatter, grid, dim3(kBinThreads), lds, st, a.prect, a.depth, a.P, per, a.TX, local,
                       (const uint32_t*)a.counts, a.cap, a.ent);
}

}  // namespace dgs
