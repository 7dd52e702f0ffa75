// Stable LSD radix sort of (key, u32 value) pairs, 8-bit digits, for u32 and
// u64 keys and any run of digits [first_bit, first_bit + bits), first_bit a multiple of 8.
//
// Each pass counts, then scatters.  k_sort_count counts the pass's digit in
// every partition of the keys; k_sort_scan turns the table [partition][digit]
// into each partition's offset within the digit and the digits' totals;
// k_sort_scatter ranks a partition's keys stably (wavefront ballots match
// equal digits) and writes them digit-grouped from LDS, so that every store
// covers a contiguous run.  No workgroup waits for another.  With one sweep
// per pass whose partitions handed their counts on by look-back, the hops over
// a thousand partitions were most of a pass: 4,000,037 pairs of 64-bit keys
// took 56 us a pass and 58 us for the digit counts of all passes, 450 us for
// 47 bits; count, scan and scatter are 6.2 + 4.9 + 18.5 us a pass, 223 us in
// all, with 21 us for a pass's 96 MB at the copy rate.
// The key count is read on the device: a frame needs no host round trip.
#include "common.h"
#include "launch.h"

namespace dgs {

// Partitions of 4096 keys in workgroups of 512 threads: 39 KB of LDS and at
// most 64 registers, so that four share a CU and all of 4 M keys' partitions
// are resident at once.  Sorts of fewer than 2^19 keys, which would leave half
// of the CUs idle, take partitions of 1024 in workgroups of 256 threads
// (47-bit sorts of 250,000 and 500,000 keys: 93 and 107 us, 110 and 121 with
// the large partitions).  The size is chosen on the host, by the key count of a
// caller's sort and of a frame's depth sort, by the capacity of its key sort (at
// least 2^20 unless reserved smaller).
constexpr int kSmallPart = 1024;
constexpr int64_t kSmallSort = (int64_t)1 << 19;
// A table of at most this many rows is summed by the scatter itself: 47-bit
// sorts of 20,000 and 60,000 keys 76 and 83 us, 84 and 86 with the scan's
// launch; with 256 rows 250,000 keys take 135 us instead of 93.
constexpr uint32_t kDirectParts = 64;
constexpr int kScanDigits = 16;   // digits per workgroup of the table's scan: one 64-byte line of each row
constexpr int kScanRowLanes = 1024 / kScanDigits;
constexpr int kScanRows = 16;     // rows per thread and step

int sort_passes(int bits) { return (bits + 7) / 8; }

static size_t max_parts(int64_t cap) { return (size_t)((cap + kSmallPart - 1) / kSmallPart); }

size_t sort_status_words(int64_t cap) { return max_parts(cap) * 256; }

// The grid of a frame's sort is for the capacity, of which it may use little:
// beyond this many workgroups they take several partitions each.  A 1920 x 1080
// frame of 546,000 keys in a buffer of 2^28 took 490 us, 131 of them in two
// passes of 65,536 workgroups nearly all without keys; now 390, 377 with 4096
// workgroups, which a frame of 54 M keys pays for (2100 us, with 4096 2212).
constexpr uint32_t kMaxGrid = 16384;

// Partition i of the workgroups' order: each XCD (block % 8) has one contiguous
// range of them, so that the runs which neighbouring partitions write into one
// line meet in that XCD's L2.  nparts or more: none.
__device__ __forceinline__ uint32_t nth_part(uint32_t i, uint32_t nparts) {
    const uint32_t per = (nparts + kXcds - 1) / kXcds, k = i / kXcds;
    return k < per ? i % kXcds * per + k : nparts;
}

// Digit of a key at a shift that is a multiple of 8: it lies in one word.
__device__ __forceinline__ uint32_t digit(uint64_t k, int shift) {
    return ((shift < 32 ? (uint32_t)k : (uint32_t)(k >> 32)) >> (shift & 31)) & 255u;
}
__device__ __forceinline__ uint32_t digit(uint32_t k, int shift) { return (k >> shift) & 255u; }

// Runs f(part) for the workgroup's partitions (LOOP: several).
template <bool LOOP, class F>
__device__ __forceinline__ void own_parts(uint32_t nparts, F f) {
    uint32_t b = blockIdx.x;
    for (;;) {
        const uint32_t part = nth_part(b, nparts);
        if (part >= nparts) return;
        f(part);
        if (!LOOP) return;
        __syncthreads();  // the LDS is written again
        b += gridDim.x;
    }
}

template <class KeyT, int THREADS, int ITEMS, bool LOOP>
__global__ __launch_bounds__(THREADS) void k_sort_count(const KeyT* __restrict__ keys,
                                                        const uint32_t* __restrict__ n_ptr, uint32_t cap, int shift,
                                                        uint32_t* __restrict__ counts) {
    constexpr uint32_t kPart = THREADS * ITEMS;
    constexpr int kCopies = 4;
    __shared__ uint32_t s_cnt[kCopies][256];
    const uint32_t tid = threadIdx.x;
    uint32_t* cnt = s_cnt[(tid >> 6) % kCopies];
    uint32_t n = n_ptr ? *n_ptr : cap;
    if (n > cap) n = cap;
    const uint32_t nparts = (n + kPart - 1) / kPart;
    own_parts<LOOP>(nparts, [&](uint32_t part) __attribute__((always_inline)) {
        const uint32_t pbase = part * kPart;
        KeyT k[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const uint32_t idx = pbase + i * THREADS + tid;
            k[i] = keys[idx < n ? idx : n - 1];
        }
        for (uint32_t d = tid; d < kCopies * 256; d += THREADS) (&s_cnt[0][0])[d] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; i++)
            if (pbase + i * THREADS + tid < n) atomicAdd(&cnt[digit(k[i], shift)], 1u);
        __syncthreads();
        if (tid < 256) {
            uint32_t s = 0;
#pragma unroll
            for (int c = 0; c < kCopies; c++) s += s_cnt[c][tid];
            counts[(size_t)part * 256 + tid] = s;
        }
    });
}

// Columns of the table [partition][digit] -> exclusive prefixes, in place;
// totals[digit] = the column's sum.
__global__ __launch_bounds__(1024) void k_sort_scan(uint32_t* __restrict__ counts, const uint32_t* __restrict__ n_ptr,
                                                    uint32_t cap, uint32_t part_keys, uint32_t* __restrict__ totals) {
    __shared__ uint32_t s_sum[16][kScanDigits];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t dl = tid % kScanDigits, d = blockIdx.x * kScanDigits + dl, rl = tid / kScanDigits;
    uint32_t n = n_ptr ? *n_ptr : cap;
    if (n > cap) n = cap;
    const uint32_t nparts = (n + part_keys - 1) / part_keys;
    uint32_t carry = 0;
    for (uint32_t r0 = 0; r0 < nparts; r0 += kScanRowLanes * kScanRows) {
        const uint32_t row = r0 + rl * kScanRows;
        uint32_t c[kScanRows], sum = 0;
#pragma unroll
        for (int i = 0; i < kScanRows; i++) c[i] = row + i < nparts ? counts[(size_t)(row + i) * 256 + d] : 0u;
#pragma unroll
        for (int i = 0; i < kScanRows; i++) sum += c[i];
        // inclusive over the wavefront's four row lanes, then over the wavefronts
        uint32_t x = sum, u = __shfl_up(x, 16, 64);
        if (lane >= 16) x += u;
        u = __shfl_up(x, 32, 64);
        if (lane >= 32) x += u;
        if (lane >= 48) s_sum[wave][dl] = x;
        __syncthreads();
        uint32_t pre = carry;
#pragma unroll
        for (uint32_t w = 0; w < 16; w++) {
            const uint32_t s = s_sum[w][dl];
            if (w < wave) pre += s;
            carry += s;
        }
        uint32_t run = pre + x - sum;
#pragma unroll
        for (int i = 0; i < kScanRows; i++) {
            if (row + i < nparts) counts[(size_t)(row + i) * 256 + d] = run;
            run += c[i];
        }
        __syncthreads();  // s_sum is written again
    }
    if (rl == 0) totals[d] = carry;
}

// Number of set bits of `mask` at lanes below this one.
__device__ inline uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// n_ptr (device) holds the item count, or is null for n = cap.  DIRECT: counts
// holds the partitions' counts (at most kDirectParts rows), else their
// prefixes, and totals the digits' totals.
template <class KeyT, int THREADS, int ITEMS, bool DIRECT, bool LOOP>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(THREADS == 512 ? 8 : 1)))
void k_sort_scatter(const KeyT* __restrict__ kin, const uint32_t* __restrict__ vin, KeyT* __restrict__ kout,
                    uint32_t* __restrict__ vout, const uint32_t* __restrict__ n_ptr, uint32_t cap, int shift,
                    const uint32_t* __restrict__ counts, const uint32_t* __restrict__ totals) {
    constexpr uint32_t kPart = THREADS * ITEMS;
    constexpr int kWaves = THREADS / 64;
    static_assert(ITEMS * 64 < 65536 && kPart < 65536, "16-bit counters");
    __shared__ KeyT s_key[kPart];         // the keys, then the values, in digit order
    __shared__ uint16_t s_cnt[kWaves][256];  // per-wave digit counts, then per-wave offsets
    __shared__ uint32_t s_lstart[256];    // start of each digit in the partition's order
    __shared__ uint32_t s_gbase[256];     // global start of each digit's run minus its local start
    __shared__ uint32_t s_wsum[2][4];
    uint32_t* s_val = reinterpret_cast<uint32_t*>(s_key);
    uint32_t n = n_ptr ? *n_ptr : cap;
    if (n > cap) n = cap;
    const uint32_t nparts = (n + kPart - 1) / kPart;
    own_parts<LOOP>(nparts, [&](uint32_t part) __attribute__((always_inline)) {
        uint32_t tid = threadIdx.x;
        if (LOOP) asm volatile("" : "+v"(tid));  // nothing made of it is kept from part to part in registers
        const uint32_t lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const uint32_t pbase = part * kPart, wbase = pbase + wave * (ITEMS * 64);  // uniform
        const uint32_t left = n > wbase ? n - wbase : 0u;  // keys from the wavefront's first on
        // a lane past the end reads the last key again (a wavefront past it key 0)
        const uint32_t rmax = left ? left - 1 : 0u;
        const KeyT* kw = kin + (left ? wbase : 0u);
        const uint32_t* vw = vin + (left ? wbase : 0u);
        KeyT k[ITEMS];
        uint32_t v[ITEMS], rank[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; i++) k[i] = kw[min(i * 64 + lane, rmax)];
        uint32_t excl = 0, total = 0;
        if (DIRECT) {
            if (tid < 256 && nparts > 1)
#pragma unroll 8
                for (uint32_t r = 0; r < nparts; r++) {
                    const uint32_t c = counts[r * 256 + tid];
                    total += c;
                    excl += r < part ? c : 0u;
                }
        } else if (tid < 256) {
            excl = counts[(size_t)part * 256 + tid];
            total = totals[tid];
        }
        for (uint32_t d = tid; d < kWaves * 128; d += THREADS) reinterpret_cast<uint32_t*>(s_cnt)[d] = 0;
        __syncthreads();
        // stable ranking inside the wave: item i of every lane precedes item i+1
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const bool valid = i * 64 + lane < left;
            const uint32_t d = digit(k[i], shift);
            // lanes whose digit differs, bit by bit; lanes without a key differ
            const uint64_t vb = __ballot(valid);
            uint32_t dlo = ~(uint32_t)vb, dhi = ~(uint32_t)(vb >> 32);
#pragma unroll
            for (int b = 0; b < 8; b++) {
                const uint32_t m = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // all ones where the bit is set
                const uint64_t bb = __ballot(m != 0);
                dlo |= (uint32_t)bb ^ m;
                dhi |= (uint32_t)(bb >> 32) ^ m;
            }
            const uint64_t peers = ~((uint64_t)dhi << 32 | dlo);
            uint32_t before = 0;
            if (valid) before = s_cnt[wave][d];
            rank[i] = before + lanes_below(peers);
            asm volatile("" : "+v"(rank[i]));  // now: kept as its three operands, the ranks spill
            if (valid && lane == (uint32_t)__builtin_ctzll(peers))
                s_cnt[wave][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int i = 0; i < ITEMS; i++) v[i] = vw[min(i * 64 + lane, rmax)];
        __syncthreads();
        // thread d < 256: digit d's per-wave offsets, its start in the
        // partition and in the output
        uint32_t tot = 0, x = 0, y = 0;
        if (tid < 256) {
#pragma unroll
            for (int w = 0; w < kWaves; w++) {
                const uint32_t c = s_cnt[w][tid];
                s_cnt[w][tid] = (uint16_t)tot;
                tot += c;
            }
            if (DIRECT && nparts == 1) total = tot;  // the only partition: nothing was counted before
            x = tot;
            y = total;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = __shfl_up(x, o, 64), t = __shfl_up(y, o, 64);
                if (lane >= (uint32_t)o) {
                    x += u;
                    y += t;
                }
            }
            if (lane == 63) {
                s_wsum[0][wave] = x;
                s_wsum[1][wave] = y;
            }
        }
        __syncthreads();
        if (tid < 256) {
            uint32_t lstart = x - tot, gstart = y - total;
            for (uint32_t w = 0; w < wave; w++) {
                lstart += s_wsum[0][w];
                gstart += s_wsum[1][w];
            }
            s_lstart[tid] = lstart;
            s_gbase[tid] = gstart + excl - lstart;
        }
        __syncthreads();
        // the partition in digit order through LDS: keys, then values
#pragma unroll
        for (int i = 0; i < ITEMS; i++)
            if (i * 64 + lane < left) {
                const uint32_t d = digit(k[i], shift);
                rank[i] += s_lstart[d] + s_cnt[wave][d];
                s_key[rank[i]] = k[i];
            }
        __syncthreads();
        const uint32_t cnt = n - pbase < kPart ? n - pbase : kPart;
        uint32_t pos[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
            const uint32_t j = tid + i * THREADS;
            pos[i] = n;
            if (j < cnt) {
                const KeyT kk = s_key[j];
                pos[i] = s_gbase[digit(kk, shift)] + j;
                // below n, unless the caller's keys changed under the sort
                if (pos[i] < n) kout[pos[i]] = kk;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; i++)
            if (i * 64 + lane < left) s_val[rank[i]] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; i++)
            if (pos[i] < n) vout[pos[i]] = s_val[tid + i * THREADS];
    });
}

template <class KeyT, int THREADS, int ITEMS>
static void sort_passes_launch(hipStream_t st, KeyT* k0, uint32_t* v0, KeyT* k1, uint32_t* v1,
                               const uint32_t* n_ptr, uint32_t cap, int first_bit, int passes, const SortScratch& s) {
    constexpr uint32_t kPart = THREADS * ITEMS;
    const uint32_t parts = (uint32_t)(((uint64_t)cap + kPart - 1) / kPart);
    const uint32_t groups = (parts + kXcds - 1) / kXcds * kXcds;
    const bool loop = n_ptr && groups > kMaxGrid;
    const dim3 grid(loop ? kMaxGrid : groups), block(THREADS);
    KeyT *ki = k0, *ko = k1;
    uint32_t *vi = v0, *vo = v1;
    for (int p = 0; p < passes; p++) {
        const int shift = first_bit + 8 * p;
        const auto launch = [&](auto* count, auto* scatter, bool direct) {
            if (parts > 1) hipLaunchKernelGGL(count, grid, block, 0, st, ki, n_ptr, cap, shift, s.counts);
            if (!direct)
                hipLaunchKernelGGL(k_sort_scan, dim3(256 / kScanDigits), dim3(1024), 0, st, s.counts, n_ptr, cap, kPart,
                                   s.totals);
            hipLaunchKernelGGL(scatter, grid, block, 0, st, ki, vi, ko, vo, n_ptr, cap, shift, s.counts, s.totals);
        };
        if (parts <= kDirectParts)
            launch(k_sort_count<KeyT, THREADS, ITEMS, false>, k_sort_scatter<KeyT, THREADS, ITEMS, true, false>, true);
        else if (!loop)
            launch(k_sort_count<KeyT, THREADS, ITEMS, false>, k_sort_scatter<KeyT, THREADS, ITEMS, false, false>, false);
        else if constexpr (THREADS == 512)  // sorts with small partitions have few of them
            launch(k_sort_count<KeyT, THREADS, ITEMS, true>, k_sort_scatter<KeyT, THREADS, ITEMS, false, true>, false);
        KeyT* tk = ki; ki = ko; ko = tk;
        uint32_t* tv = vi; vi = vo; vo = tv;
    }
}

template <class KeyT>
static bool radix_sort(hipStream_t st, KeyT* k0, uint32_t* v0, KeyT* k1, uint32_t* v1, const uint32_t* n_ptr,
                       uint32_t cap, int first_bit, int bits, const SortScratch& s) {
    const int passes = sort_passes(bits);
    if (passes <= 0 || cap == 0) return false;
    if (cap < kSmallSort)
        sort_passes_launch<KeyT, 256, kSmallPart / 256>(st, k0, v0, k1, v1, n_ptr, cap, first_bit, passes, s);
    else
        sort_passes_launch<KeyT, 512, 8>(st, k0, v0, k1, v1, n_ptr, cap, first_bit, passes, s);
    return (passes & 1) != 0;
}

bool launch_radix_sort(hipStream_t st, uint64_t* k0, uint32_t* v0, uint64_t* k1, uint32_t* v1,
                       const uint32_t* n_ptr, uint32_t cap, int bits, const SortScratch& s, int first_bit) {
    return radix_sort(st, k0, v0, k1, v1, n_ptr, cap, first_bit, bits, s);
}

bool launch_radix_sort32(hipStream_t st, uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, uint32_t n,
                         const SortScratch& s) {
    return radix_sort(st, k0, v0, k1, v1, nullptr, n, 0, 32, s);
}

}  // namespace dgs
