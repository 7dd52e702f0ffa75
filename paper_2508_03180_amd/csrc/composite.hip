// Tile compositors.
//
// Duplex (Sec. V-A, eq. hybrid_renderer with w_n = v_n T_n, eq. dulpex_T;
// Sec. V-B early termination; Sec. VI-A false-positive skip).  For every
// pixel the cells of its tile are walked front to back.  Inside a cell the
// members are summed without order:
//     A = sum alpha c,  B = sum alpha,  P = prod (1 - v alpha)
// over members whose box contains the pixel and whose alpha reaches
// alpha_min, with alpha = min(alpha_max, sigma G'(x')).  Across cells
//     N += v T A,  D += v T B,  T *= P,
// a cell is blended only while T (the transmittance in front of it) is at
// least eps, and the colour is C = N / D (bg where D = 0).
//
// Alpha (eqs. alpha_blending, transmittance): the same walk over
// depth-sorted Gaussians with C += T alpha c, T *= 1 - alpha, plus T bg.
//
// Mapping: a wavefront runs without workgroup barriers and owns a whole 16x16
// tile or, for tiles with long lists, a 16x8 half or an 8x8 quarter of it (a
// Block of 4, 2 or 1 strips of 64 pixels; lane l holds one pixel of every
// strip it owns).  Work items are taken
// from a queue that lists them heaviest first.  The tile list is consumed in
// chunks of up to 64 Gaussian records (whole cells): each lane loads one
// record, the wave ballots which strips every record's box touches, and the
// records go to the wave's private LDS slot, from which they are read as
// broadcasts.  The next chunk is fetched into registers while the current
// one is composited.  Cells and members that touch none of the tile's
// strips are skipped with scalar bit tests on the ballots.
#include "cells.h"
#include "common.h"
#include "launch.h"
#include "order.h"

namespace dgs {

constexpr int kWaves = 4;  // tiles per workgroup


struct Chunk {
    float4 r0, r1, r2;  // this lane's record
    float v;            // v of this lane's cell (Duplex walks)
    bool ok;
    int nch;            // entries in the chunk (cells, or Gaussians in the alpha walk)
    int first, cnt;     // cell walks, lane c < nch: first record lane and member count of cell c
};

// The next chunk of a cell walk: whole cells from list position pos (at
// most 64 records, at most end - pos cells).
template <bool RAGGED>
__device__ inline void load_cell_chunk(const CompositeArgs& a, uint32_t pos, uint32_t end, int lane, Chunk& q) {
    // every field is set on every path: a partly set struct would be kept in
    // scratch memory instead of registers
    CellChunk ch;
    load_cells<RAGGED>(a.vals, a.offs, a.cell_v, a.K, pos, end, -1, lane, ch);
    q.nch = ch.nch;
    q.first = ch.first;
    q.cnt = ch.cnt;
    q.ok = ch.g >= 0;
    q.v = ch.v;
    q.r0 = q.r1 = q.r2 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (!q.ok) return;
    const float4* p = reinterpret_cast<const float4*>(a.recs + ch.g);
    q.r0 = p[0];
    q.r1 = p[1];
    q.r2 = p[2];
}

// The next chunk of the per-Gaussian walk: up to 64 list entries from pos,
// whose ids are at hand (id: this lane's).
__device__ inline void load_gauss_chunk(const CompositeArgs& a, uint32_t pos, uint32_t end, int lane, uint32_t id, Chunk& q) {
    const int n = (int)min(64u, end - pos);
    q.nch = n;
    q.first = q.cnt = 0;
    q.ok = lane < n;
    q.r0 = q.r1 = q.r2 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    q.v = 0.0f;
    if (!q.ok) return;
    const float4* p = reinterpret_cast<const float4*>(a.recs + id);
    q.r0 = p[0];
    q.r1 = p[1];
    q.r2 = p[2];
}

// What a record's box covers of the block: its columns (bit x for column bx + x),
// for a quarter its pixels (the bit of each one's lane).  Nothing when it misses
// the block.
template <int NS>
struct BoxCover {
    uint32_t cols = 0;
    // may the record hit one of the pixels `am` (lanes of a strip that it touches)?
    __device__ __forceinline__ bool meets(uint64_t am) const { return (cols & active_columns<NS>(am)) != 0u; }
};
// A quarter's 64 pixels are one strip: by columns alone, records below a skyline
// met the sky's pixels above them, which blend to the list's end (64 x 227 pixels
// of a street view, 74,000 cells of 11: frame 2373 -> 1657 us).
template <>
struct BoxCover<1> {
    uint32_t lo = 0, hi = 0;
    __device__ __forceinline__ bool meets(uint64_t am) const {
        return ((lo & (uint32_t)am) | (hi & (uint32_t)(am >> 32))) != 0u;
    }
};

// Ballots of the owned strips each lane's record touches: B[j] for strip j of
// the block.  The block's origin is wavefront-uniform, so the ballots stay in
// scalar registers.
// Also returns, per lane, what its record's box covers.
template <int NS>
__device__ inline void strip_ballots(const Chunk& q, int bx, int by, uint64_t* B, BoxCover<NS>& box) {
    constexpr int W = Block<NS>::kCols, R = Block<NS>::kRows;
    uint32_t sm = 0;  // strip bits
    box = BoxCover<NS>();
    if (q.ok) {
        const int x0 = __float_as_int(q.r2.y), y0 = __float_as_int(q.r2.z);
        const uint32_t wxy = __float_as_uint(q.r2.w);
        const int x1 = x0 + (int)(wxy & 0xffffu), y1 = y0 + (int)(wxy >> 16);
        if (x0 <= bx + W - 1 && x1 >= bx) {
            const int lo = max(x0, bx) - bx, hi = min(x1, bx + W - 1) - bx;
            const uint32_t cols = ((2u << (hi - lo)) - 1u) << lo;
#pragma unroll
            for (int j = 0; j < NS; j++) {
                const int r0 = by + R * j;
                if (y0 <= r0 + R - 1 && y1 >= r0) sm |= 1u << j;
            }
            if constexpr (NS == 1) {
                if (sm) {
                    const int first = max(y0, by) - by, last = min(y1, by + R - 1) - by;
                    const uint64_t rows = (~0ull >> (56 - 8 * last)) & (~0ull << (8 * first));
                    box.lo = cols * 0x01010101u & (uint32_t)rows;
                    box.hi = cols * 0x01010101u & (uint32_t)(rows >> 32);
                }
            } else {
                box.cols = cols;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NS; j++) B[j] = __ballot((sm >> j) & 1u);
}

__device__ inline void store_chunk(GRec* lds, int lane, const Chunk& q) {
    if (!q.ok) return;
    float4* d = reinterpret_cast<float4*>(lds + lane);
    d[0] = q.r0;
    d[1] = q.r1;
    d[2] = q.r2;
}

struct RecView {
    float ox, oy, ca, cb, cc, lo, r, g, b;
    int x0, y0;
    uint32_t wx, wy;
};

typedef float F4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const F4 LdsF4;

// The wavefront's record array as a 32-bit LDS address, held in a scalar
// register: every lane reads the same record, so its address is uniform.
__device__ inline uint32_t lds_base(const GRec* lds) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const LdsF4*)lds);
}

__device__ inline RecView read_rec(uint32_t lb, int i) {
    const LdsF4* p = (const LdsF4*)(uintptr_t)(lb + (uint32_t)i * (uint32_t)sizeof(GRec));
    const F4 a = p[0], b = p[1], c = p[2];
    RecView e;
    e.ox = a.x; e.oy = a.y; e.ca = a.z; e.cb = a.w;
    e.cc = b.x; e.lo = b.y; e.r = b.z; e.g = b.w;
    e.b = c.x;
    e.x0 = __float_as_int(c.y);
    e.y0 = __float_as_int(c.z);
    const uint32_t wxy = __float_as_uint(c.w);
    e.wx = wxy & 0xffffu;
    e.wy = wxy >> 16;
    return e;
}


// The frame's values the compositors use, loaded once per wavefront from the
// device frame record (scalar registers; the kernel argument is left as is).
// The output pointers are global-memory pointers: stored through generic
// pointers, they became flat stores, which the compiler counts as possible
// LDS accesses too, so every later wait for an LDS read had to wait for all
// of them.
typedef __attribute__((address_space(1))) float GFloat;
typedef __attribute__((address_space(1))) int32_t GInt;
struct FrameView {
    int TX, W, H;
    float eps, th, amax, bg0, bg1, bg2;
    GFloat* color;
    GFloat* D;
    GFloat* T;
    GInt* last;
    GFloat* sv_color;  // saved state of the frame for its backward (SAVE walks only)
    GFloat* sv_D;
    GFloat* sv_T;
    GInt* sv_last;
};

__device__ inline FrameView frame_view(const FrameK* fr) {
    FrameView f;
    f.TX = fr->k.TX;
    f.W = fr->k.W;
    f.H = fr->k.H;
    f.eps = fr->o.no_et ? 0.0f : fr->o.eps;
    f.th = fr->o.log2_alpha_min;
    f.amax = fr->o.alpha_max;
    f.bg0 = fr->o.bg[0];
    f.bg1 = fr->o.bg[1];
    f.bg2 = fr->o.bg[2];
    f.color = (GFloat*)fr->color;
    f.D = (GFloat*)fr->D;
    f.T = (GFloat*)fr->T;
    f.last = (GInt*)fr->last;
    f.sv_color = (GFloat*)fr->sv_color;
    f.sv_D = (GFloat*)fr->sv_D;
    f.sv_T = (GFloat*)fr->sv_T;
    f.sv_last = (GInt*)fr->sv_last;
    return f;
}

// Work item: tile << 3 | mode; mode 0 = the whole tile (all four strips),
// mode 2 + h = half h, mode 4 + q = quarter q (a Block of 4, 2 or 1 strips).

// Statistics counters (STATS only): n_val, n_rendered (the termination ratio
// 1 - n_rendered / n_val), in-box member evaluations and (pixel, entry) pairs
// that contributed, for the algorithmic work count.
struct Counters {
    uint32_t val = 0, rend = 0, box = 0, cellhit = 0, cellpx = 0;
};

// The hybrid renderer over one tile (NS = 4), half (2) or quarter (1)
// (Sec. V-A, eq. hybrid_renderer with w_n = v_n T_n and eq. dulpex_T; Sec. V-B
// termination; Sec. VI-A box gate): cells front to back; a pixel whose
// transmittance in front of a cell is below eps stops there; inside a cell
// every member that passes the box and alpha_min gates adds w alpha c to N
// and w alpha to D with the cell's weight w = v T (the cell's alpha sums A,
// B of the equation times w, accumulated member by member), and
// P = prod (1 - v alpha) updates T after the cell; C = N / D at the end.
// LC: the "w/o T^cell" weights -- cell_v holds w_n = v_n max(0, 1 - d_n / tau),
// no transmittance and no termination.
// A cell counts as contributing at a pixel (`last`) when any of its members
// passed both gates there, whatever its weight.
// SAVE: also write the state the backward replays from -- colour, D, and the
// list position of the last contributing cell whose transmittance in front
// is at least kMinReplayT together with that transmittance.
// RAGGED: cells with their own member counts (CSR offsets), else K per cell.
template <bool STATS, int NS, bool LC, bool SAVE, bool RAGGED>
__device__ inline void duplex_tile(const CompositeArgs& a, const FrameView& f, int tile, int part, int lane, GRec* lds,
                                 Counters& cn) {
    const Block<NS> bl((tile % f.TX) * kTile, (tile / f.TX) * kTile, part);
    const int px = bl.x + Block<NS>::column(lane), py0 = bl.y + Block<NS>::row(lane);
    const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
    // a quarter's rows: offsets from the row shift above (row_shift)
    const int shift = NS == 1 ? row_shift(py0 & (kTile - 1), end - start, kSplitLenCells) : 0;
    const float shiftf = (float)shift;
    const int K = a.K;
    const uint32_t kmask = member_mask(K);
    const float eps = f.eps, th = f.th, amax = f.amax;
    const uint32_t lb = lds_base(lds);

    float T[NS], N0[NS], N1[NS], N2[NS], D[NS];
    float thj[NS];  // gate threshold of strip j's pixel for the current cell, +inf once it has terminated
    int32_t last[NS];
    int32_t rlast[NS];  // SAVE: replay start (list position + 1, 0 = none)
    float rT[NS];       // SAVE: transmittance in front of that entry
    bool inb[NS];  // the pixel lies in the image
#pragma unroll
    for (int j = 0; j < NS; j++) {
        T[j] = 1.0f; N0[j] = N1[j] = N2[j] = D[j] = 0.0f; last[j] = 0;
        rlast[j] = 0; rT[j] = 1.0f;
        inb[j] = px < f.W && py0 + 4 * j < f.H;
        thj[j] = inb[j] ? th : INFINITY;
    }
    // the per-cell ballots below are ballots of single compares, combined
    // with these as scalar masks (a ballot of a combination of lane masks
    // is rebuilt through a vector register first)
    uint64_t inbm[NS];  // strip j's pixels in the image
#pragma unroll
    for (int j = 0; j < NS; j++) inbm[j] = __ballot(inb[j]);

    Chunk q;
    if (start < end) load_cell_chunk<RAGGED>(a, start, end, lane, q);
    bool alive = true;
    for (uint32_t pos = start; pos < end && (alive || STATS);) {
        const int nch = q.nch;
        int cfirst = 0, ccnt = 0;  // of this chunk (q takes the next one below)
        if constexpr (RAGGED) {
            cfirst = q.first;
            ccnt = q.cnt;
        }
        // Duplex: log2 v goes into the record's log2 sigma, so that the
        // walk computes v alpha directly (the alpha_min test moves by log2 v)
        // per record lane, its cell's gate threshold and weight clamp (read
        // by the cell loop from the cell's first lane)
        float cthc = th, cvmax = amax;
        if (!LC) {
            const float lv = fold_log2_weight(q.v);
            q.r1.y += lv;
            cthc = th + lv;
            cvmax = q.v * amax;
        }
        store_chunk(lds, lane, q);
        uint64_t B[NS];
        BoxCover<NS> box;  // of this lane's record
        strip_ballots<NS>(q, bl.x, bl.y, B, box);
        const float cv = q.v;
        const uint32_t next = pos + nch;
        if (next < end) load_cell_chunk<RAGGED>(a, next, end, lane, q);
        for (int c = 0; c < nch; c++) {
            if (STATS) {  // (pixel, cell) pairs the walk reaches: listed, in the image, not terminated
#pragma unroll
                for (int j = 0; j < NS; j++) cn.cellpx += LC ? inb[j] : inb[j] && !(T[j] < eps);
            }
            // fixed K: cell c holds record lanes cK .. cK + K - 1
            const int base = RAGGED ? lane_value(cfirst, c) : c * K;
            const uint32_t cm = RAGGED ? member_mask(lane_value(ccnt, c)) : kmask;
            uint32_t mj[NS], any = 0;
#pragma unroll
            for (int j = 0; j < NS; j++) {
                mj[j] = (uint32_t)(B[j] >> base) & cm;
                any |= mj[j];
            }
            if (!any) continue;  // no member of this cell touches the owned strips
            const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cv), base));
            // Duplex: every record of this cell holds log2 sigma + log2 v, so
            // its power pw is log2(v sigma G'); alpha >= alpha_min becomes
            // pw >= th + log2 v and min(alpha_max, .) becomes min(v alpha_max, .)
            const float thc = LC ? th : __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cthc), base));
            const float vmax = LC ? amax : __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cvmax), base));
            // a pixel still blends while T >= eps (T never rises, so once
            // below eps it stays below: no state is carried across cells)
            bool act[NS];
#pragma unroll
            for (int j = 0; j < NS; j++) act[j] = LC ? inb[j] : inb[j] && !(T[j] < eps);
            if constexpr (!LC) {
                uint64_t am[NS], amall = 0;  // ballots of act
#pragma unroll
                for (int j = 0; j < NS; j++) {
                    thj[j] = act[j] ? thc : INFINITY;
                    am[j] = __ballot(!(T[j] < eps)) & inbm[j];
                    amall |= am[j];
                }
                if (!STATS && !amall) {
                    alive = false;
                    break;
                }
                // once pixels have terminated, a member whose box misses every
                // pixel still blending cannot change anything: drop it (a
                // finished pixel has threshold +inf, so it is never hit)
                if (!STATS) {
                    uint32_t live = 0;
#pragma unroll
                    for (int j = 0; j < NS; j++) {
                        if (am[j] == inbm[j]) {  // every pixel of strip j still blends
                            live |= mj[j];
                            continue;
                        }
                        // B[j]: the records touching strip j
                        mj[j] = (uint32_t)((__ballot(box.meets(am[j])) & B[j]) >> base) & cm;
                        live |= mj[j];
                    }
                    any = live;
                    if (!any) continue;  // no member reaches a blending pixel: T, last unchanged
                }
            }
            // the cell's weight is fixed before its members: w alpha c and
            // w alpha go straight into N and D (no per-cell sums A, B); in the
            // Duplex walk al below is v alpha and w alpha = T (v alpha)
            float wj[NS], P[NS];
            // pixels where some member of this cell passed both gates (a scalar
            // mask: a bool carried through the member loop is merged with the
            // exec mask by scalar instructions every iteration)
            uint64_t hcm[NS];
#pragma unroll
            for (int j = 0; j < NS; j++) { wj[j] = LC ? v : T[j]; P[j] = 1.0f; hcm[j] = 0; }
            const auto member = [&](const RecView& e) {
                const uint32_t rx = (uint32_t)(px - e.x0);
                const bool inx = rx <= e.wx;
                const float dx = (float)(int)rx + e.ox;
                // outside the box's columns the power is -inf: the alpha_min
                // test then rejects the pixel as the box test would
                const float t0 = inx ? fmaf(e.ca * dx, dx, e.lo) : -INFINITY;
                const float t1 = e.cb * dx;
                const uint32_t ry0 = (uint32_t)(py0 - shift - e.y0);
                const float dy0 = (float)(int)ry0 + e.oy;
                // every strip's power and gates first (strips the member misses
                // fail the row test in every lane): no scalar test per strip
                float pw[NS];
                // pixels hit: both gates, false once the pixel has terminated.  As
                // scalar masks, each the AND of ballots of single compares: the
                // cell's hit flag is then one scalar OR instead of a select
                // (1920 x 1080, 100,000 cells: 227 -> 223 us; 4K street view 381
                // -> 350).  Skipping the rest of a member that hits no pixel, by
                // a scalar test, costs more than it saves (228 and 369 us).
                uint64_t hm[NS];
#pragma unroll
                for (int j = 0; j < NS; j++) {
                    const uint32_t ry = NS == 1 ? ry0 + (uint32_t)shift : ry0 + 4u * j;
                    const float dy = NS == 1 ? dy0 + shiftf : j ? dy0 + 4.0f * j : dy0;  // the row 4j below, without a conversion
                    pw[j] = fmaf(dy, fmaf(e.cc, dy, t1), t0);
                    if (STATS) {
                        const bool iny = ry <= e.wy, val = iny & (pw[j] >= thc);
                        cn.val += val;
                        cn.rend += val && act[j];
                        cn.box += inx && iny && act[j];
                    }
                    hm[j] = __ballot(ry <= e.wy) & __ballot(pw[j] >= thj[j]);
                    hcm[j] |= hm[j];
                }
#pragma unroll
                for (int j = 0; j < NS; j++) {
                    // no branch: a pixel that is not hit adds alpha = 0, which
                    // leaves N, D and P exactly unchanged (the owned strips then
                    // interleave without exec-mask changes)
                    // min(vmax, 2^pw) as a clamp to [0, vmax] (2^pw >= 0)
                    const float al = __builtin_amdgcn_inverse_ballot_w64(hm[j])
                                         ? __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(pw[j]), 0.0f, vmax)
                                         : 0.0f;
                    const float wa = wj[j] * al;
                    N0[j] = fmaf(wa, e.r, N0[j]);
                    N1[j] = fmaf(wa, e.g, N1[j]);
                    N2[j] = fmaf(wa, e.b, N2[j]);
                    D[j] += wa;
                    if constexpr (!LC) P[j] = fmaf(-P[j], al, P[j]);
                }
            };
            // A quarter's wavefront is often alone on its SIMD (a small image
            // with long lists), where a member waits for its record and each
            // instruction for the one before it: four members at a time,
            // records read together, their powers interleaved (114 x 60 pixels,
            // 11,187 cells of 31: frame 1648 -> 1290 us, pairs alone 1453; 98 x
            // 863, 3,190 of 9: 393 -> 328).  Halves and whole tiles share their
            // SIMDs: pairs of members gain nothing there (1920 x 1080 323 us for 320).
            uint32_t rem = any;
            if constexpr (NS == 1) {
                while (__builtin_popcount(rem) >= 4) {
                    RecView e[4];
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        e[i] = read_rec(lb, base + __builtin_ctz(rem));
                        rem &= rem - 1;
                    }
#pragma unroll
                    for (int i = 0; i < 4; i++) member(e[i]);
                }
                while (rem & (rem - 1)) {
                    const RecView e0 = read_rec(lb, base + __builtin_ctz(rem));
                    rem &= rem - 1;
                    const RecView e1 = read_rec(lb, base + __builtin_ctz(rem));
                    rem &= rem - 1;
                    member(e0);
                    member(e1);
                }
            }
            for (; rem; rem &= rem - 1) member(read_rec(lb, base + __builtin_ctz(rem)));
            // no branch: a pixel that no longer blends had threshold +inf in
            // this cell, so P = 1 and no hit there (T and last unchanged)
#pragma unroll
            for (int j = 0; j < NS; j++) {
                if (!mj[j]) continue;  // scalar: nothing of this cell in strip j
                const int32_t idx = (int32_t)(pos + c - start + 1);
                const bool hc = __builtin_amdgcn_inverse_ballot_w64(hcm[j]);
                if constexpr (SAVE) {
                    const bool rep = hc && T[j] >= kMinReplayT;
                    rlast[j] = rep ? idx : rlast[j];
                    rT[j] = rep ? T[j] : rT[j];
                }
                if constexpr (!LC) T[j] *= P[j];
                last[j] = hc ? idx : last[j];
                if (STATS) cn.cellhit += hc;
            }
        }
        // a cell that touches the strips checks whether a pixel still blends; a
        // quarter may be opaque after the last one that does (8 opaque cells before
        // 12,500 entries in the tile's other quarters: 1172 us of compositor, now
        // 10).  Halves see twice the cells, and the check slows their walk.
        if (NS == 1 && !STATS && !LC) alive = alive && (__ballot(!(T[0] < eps)) & inbm[0]) != 0;
        pos = next;
    }
    const size_t HW = (size_t)f.W * f.H;
#pragma unroll
    for (int j = 0; j < NS; j++) {
        const int py = py0 + 4 * j;
        if (px >= f.W || py >= f.H) continue;
        const size_t p = (size_t)py * f.W + px;
        if (D[j] > 0.0f) {
            const float inv = 1.0f / D[j];
            f.color[p] = N0[j] * inv;
            f.color[HW + p] = N1[j] * inv;
            f.color[2 * HW + p] = N2[j] * inv;
        } else {
            f.color[p] = f.bg0;
            f.color[HW + p] = f.bg1;
            f.color[2 * HW + p] = f.bg2;
        }
        if (f.D) f.D[p] = D[j];
        if (f.T) f.T[p] = T[j];
        if (f.last) f.last[p] = last[j];
        if constexpr (SAVE) {
            f.sv_color[p] = f.color[p];
            f.sv_color[HW + p] = f.color[HW + p];
            f.sv_color[2 * HW + p] = f.color[2 * HW + p];
            f.sv_D[p] = D[j];
            f.sv_T[p] = rT[j];
            f.sv_last[p] = rlast[j];
        }
    }
}

template <bool STATS, int NS>
__device__ inline void alpha_tile(const CompositeArgs& a, const FrameView& f, int tile, int part, int lane, GRec* lds,
                                 Counters& cn) {
    const Block<NS> bl((tile % f.TX) * kTile, (tile / f.TX) * kTile, part);
    const int px = bl.x + Block<NS>::column(lane), py0 = bl.y + Block<NS>::row(lane);
    const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
    // a quarter's rows: offsets from the row shift above (row_shift)
    const int shift = NS == 1 ? row_shift(py0 & (kTile - 1), end - start, kSplitLenGauss) : 0;
    const float shiftf = (float)shift;
    const float eps = f.eps, th = f.th, amax = f.amax;

    float T[NS], C0[NS], C1[NS], C2[NS];
    int32_t last[NS];
    bool inb[NS];  // the pixel lies in the image
#pragma unroll
    for (int j = 0; j < NS; j++) {
        T[j] = 1.0f; C0[j] = C1[j] = C2[j] = 0.0f; last[j] = 0;
        inb[j] = px < f.W && py0 + 4 * j < f.H;
    }
    uint64_t inbm[NS];  // strip j's pixels in the image (ballots of single compares below)
#pragma unroll
    for (int j = 0; j < NS; j++) inbm[j] = __ballot(inb[j]);
    const uint32_t lb = lds_base(lds);
    Chunk q;
    // ids are loaded two chunks ahead, records one, so that the records' addresses
    // do not wait for memory: a quarter walks a chunk in less than the two trips
    // take (105 x 57 pixels, 984,000 Gaussians: frame 3258 -> 3010 us; 1920 x 1080,
    // 1 M: 461 -> 454)
    uint32_t id = 0;
    if (start < end) {
        const uint32_t first = a.vals[min(start + lane, end - 1)];
        id = a.vals[min(start + 64 + lane, end - 1)];
        load_gauss_chunk(a, start, end, lane, first, q);
    }
    bool alive = true;
    for (uint32_t pos = start; pos < end && (alive || STATS);) {
        const int n = q.nch;
        store_chunk(lds, lane, q);
        uint64_t B[NS], any = 0;
        BoxCover<NS> box;  // of this lane's record
        strip_ballots<NS>(q, bl.x, bl.y, B, box);
#pragma unroll
        for (int j = 0; j < NS; j++) any |= B[j];
        // a quarter's termination once per chunk, however few of its records touch
        // it: where 8 of each 64 entries did, all 12,500 of a list were walked
        // after the first ones were opaque (115 us of compositor, now 10)
        if (NS == 1 && !STATS && !(__ballot(!(T[0] < eps)) & inbm[0])) break;
        const uint32_t next = pos + n;
        if (next < end) {
            load_gauss_chunk(a, next, end, lane, id, q);
            id = a.vals[min(next + 64 + lane, end - 1)];
        }
        // stops the walk when no pixel of the owned strips still blends, else
        // keeps only the records whose box meets a column that still holds a
        // blending pixel in a strip the box covers (a record outside every such
        // column and strip cannot hit a blending pixel, so dropping it changes
        // no output); false: none left
        const auto drop_finished = [&]() {
            uint64_t amall = 0, live = 0;
#pragma unroll
            for (int j = 0; j < NS; j++) {
                // every ballot runs on every lane; B[j]: the records
                // touching strip j
                const uint64_t am = __ballot(!(T[j] < eps)) & inbm[j];
                amall |= am;
                live |= __ballot(box.meets(am)) & B[j];
            }
            if (!amall) alive = false;
            any = amall ? any & live : 0;
            return any != 0;
        };
        // the gates' operands of one Gaussian, as in the Duplex walk
        struct Gate {
            float dx, t0, t1, dy0;
            uint32_t ry0;
            bool inx;
        };
        const auto gate = [&](const RecView& e) {
            Gate g;
            const uint32_t rx = (uint32_t)(px - e.x0);
            g.inx = rx <= e.wx;
            g.dx = (float)(int)rx + e.ox;
            g.t0 = g.inx ? fmaf(e.ca * g.dx, g.dx, e.lo) : -INFINITY;
            g.t1 = e.cb * g.dx;
            g.ry0 = (uint32_t)(py0 - shift - e.y0);
            g.dy0 = (float)(int)g.ry0 + e.oy;
            return g;
        };
        const auto blend = [&](int j, float pw, const RecView& e, int m) {
            const float al = fminf(amax, __builtin_amdgcn_exp2f(pw));
            const float w = al * T[j];
            C0[j] = fmaf(w, e.r, C0[j]);
            C1[j] = fmaf(w, e.g, C1[j]);
            C2[j] = fmaf(w, e.b, C2[j]);
            T[j] -= w;
            last[j] = (int32_t)(pos + m - start + 1);
            if (STATS) {
                cn.rend++;
                cn.cellhit++;
            }
        };
        if constexpr (NS == 1 && !STATS) {
            // a quarter's wavefront: four Gaussians at a time, as in the Duplex
            // walk (118 x 82 pixels, 90,000 Gaussians: frame 1308 -> 1011 us;
            // 640 x 360, 100,000: 235 -> 213); the finished ones are dropped
            // every eight
            for (int groups = 0; any; groups++) {
                if (groups && !(groups & 1) && !drop_finished()) break;
                RecView e[4];
                float pw[4];
                bool ok[4];
                int m[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const bool has = any != 0;  // none left: record 0 in its place, which hits nothing
                    m[i] = has ? __builtin_ctzll(any) : 0;
                    any &= any - 1;
                    e[i] = read_rec(lb, m[i]);
                    const Gate g = gate(e[i]);
                    const float dy = g.dy0 + shiftf;
                    pw[i] = fmaf(dy, fmaf(e[i].cc, dy, g.t1), g.t0);
                    ok[i] = has & (g.ry0 + (uint32_t)shift <= e[i].wy) & (pw[i] >= th);
                }
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (ok[i] & inb[0] & !(T[0] < eps)) blend(0, pw[i], e[i], m[i]);
            }
        } else {
            int since_check = 0;
            for (; any; any &= any - 1) {
                if (!STATS && ++since_check == 8) {
                    since_check = 0;
                    if (!drop_finished()) break;
                }
                const int m = __builtin_ctzll(any);
                const RecView e = read_rec(lb, m);
                const Gate g = gate(e);
#pragma unroll
                for (int j = 0; j < NS; j++) {
                    // termination before each Gaussian (T only changes on a hit
                    // and never rises, so no state is carried across Gaussians)
                    const bool act = inb[j] && !(T[j] < eps);
                    const uint32_t ry = NS == 1 ? g.ry0 + (uint32_t)shift : g.ry0 + 4u * j;
                    const float dy = NS == 1 ? g.dy0 + shiftf : j ? g.dy0 + 4.0f * j : g.dy0;
                    const float pw = fmaf(dy, fmaf(e.cc, dy, g.t1), g.t0);
                    const bool iny = ry <= e.wy;
                    const bool hit = iny & (pw >= th);
                    if (STATS) {
                        cn.val += hit;
                        cn.box += g.inx && iny && act;
                    }
                    if (hit & act) blend(j, pw, e, m);
                }
            }
        }
        pos = next;
    }
    const size_t HW = (size_t)f.W * f.H;
#pragma unroll
    for (int j = 0; j < NS; j++) {
        const int py = py0 + 4 * j;
        if (px >= f.W || py >= f.H) continue;
        const size_t p = (size_t)py * f.W + px;
        f.color[p] = fmaf(T[j], f.bg0, C0[j]);
        f.color[HW + p] = fmaf(T[j], f.bg1, C1[j]);
        f.color[2 * HW + p] = fmaf(T[j], f.bg2, C2[j]);
        if (f.D) f.D[p] = 1.0f - T[j];
        if (f.T) f.T[p] = T[j];
        if (f.last) f.last[p] = last[j];
    }
}

// Persistent wavefronts: each takes the next work item of a queue that lists
// them heaviest first (order.h), so long tiles start early and short ones
// fill in behind them on every XCD.  Every wavefront leaves once the queue is
// empty.
// MODE: kModeDuplex, kModeAlpha or kModeLcwsr.
template <int MODE, bool STATS, bool SAVE, bool RAGGED>
__global__ __launch_bounds__(256) void k_composite(CompositeArgs a) {
    __shared__ GRec s_rec[kWaves][64];
    const FrameView f = frame_view(a.fr);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    GRec* lds = s_rec[wave];
    const uint32_t nitems = a.queue[1];
    ItemSource src;
    Counters cn;
    // the item's number is in a scalar register: the item, its tile and its
    // half are then wavefront-uniform, and so is all loop control below
    for (uint32_t t = __builtin_amdgcn_readfirstlane(first_item<kWaves, 2>(wave, nitems, src)); t < nitems;
         t = next_item(a.queue, src, lane)) {
        const uint32_t item = a.order[t];
        const int tile = (int)(item >> 3), mode = (int)(item & 7u);
        // the costliest items, which set the kernel's span, issue ahead of the
        // others on their SIMD
        if (src.heavy)
            __builtin_amdgcn_s_setprio(3);
        else
            __builtin_amdgcn_s_setprio(0);
        if (MODE == kModeAlpha) {
            if (mode == 0)
                alpha_tile<STATS, 4>(a, f, tile, 0, lane, lds, cn);
            else if (mode >= 4)
                alpha_tile<STATS, 1>(a, f, tile, mode - 4, lane, lds, cn);
            else
                alpha_tile<STATS, 2>(a, f, tile, mode - 2, lane, lds, cn);
        } else {
            constexpr bool LC = MODE == kModeLcwsr;
            if (mode == 0)
                duplex_tile<STATS, 4, LC, SAVE, RAGGED>(a, f, tile, 0, lane, lds, cn);
            else if (mode >= 4)
                duplex_tile<STATS, 1, LC, SAVE, RAGGED>(a, f, tile, mode - 4, lane, lds, cn);
            else
                duplex_tile<STATS, 2, LC, SAVE, RAGGED>(a, f, tile, mode - 2, lane, lds, cn);
        }
    }
    if (STATS) {
        atomicAdd(&a.counters[0], (unsigned long long)cn.val);
        atomicAdd(&a.counters[1], (unsigned long long)cn.rend);
        atomicAdd(&a.counters[2], (unsigned long long)cn.box);
        atomicAdd(&a.counters[3], (unsigned long long)cn.cellhit);
        atomicAdd(&a.counters[4], (unsigned long long)cn.cellpx);
    }
}

// Builds the work queues (build_work_queue, order.h), a workgroup each.
__global__ __launch_bounds__(1024) void k_tile_order(const uint32_t* __restrict__ ranges, int ntiles,
                                                     uint32_t split_len, const uint32_t* __restrict__ total,
                                                     WorkQueue fwd, WorkQueue bwd, uint64_t* long_stat,
                                                     uint32_t prims) {
    __shared__ uint32_t s_cnt[kOrderClasses];
    __shared__ uint32_t s_part[16];
    const bool b = blockIdx.x == 1;
    build_work_queue<1024>(ranges, ntiles, b ? split_rule_bwd(split_len) : split_rule(split_len, *total),
                           b ? bwd.order : fwd.order, b ? bwd.queue : fwd.queue, s_cnt, s_part, (int)threadIdx.x,
                           b ? nullptr : long_stat, prims);
}

static unsigned persistent_grid(int tiles) {
    // enough wavefronts to fill every SIMD of the 256 CUs a few times over
    const int waves = 4 * tiles < 256 * 4 * 4 ? 4 * tiles : 256 * 4 * 4;
    return (unsigned)((waves + kWaves - 1) / kWaves);
}

void launch_tile_order(hipStream_t st, const uint32_t* ranges, int tiles, uint32_t split_len, const uint32_t* total,
                       const WorkQueue& fwd, const WorkQueue& bwd, uint64_t* long_stat, uint32_t prims) {
    if (tiles <= 0) return;
    hipLaunchKernelGGL(k_tile_order, dim3(bwd.queue ? 2 : 1), dim3(1024), 0, st, ranges, tiles, split_len, total, fwd,
                       bwd, long_stat, prims);
}

template <int MODE, bool SAVE, bool RAGGED>
static void launch_variant(hipStream_t st, dim3 g, dim3 b, const CompositeArgs& a) {
    if (a.counters)
        hipLaunchKernelGGL((k_composite<MODE, true, SAVE, RAGGED>), g, b, 0, st, a);
    else
        hipLaunchKernelGGL((k_composite<MODE, false, SAVE, RAGGED>), g, b, 0, st, a);
}

template <int MODE>
static void launch_mode(hipStream_t st, const CompositeArgs& a) {
    const int tiles = a.k.TX * a.k.TY;  // host copy of the frame's tile grid
    if (tiles <= 0) return;
    const dim3 g(persistent_grid(tiles)), b(256);
    if constexpr (MODE == kModeAlpha) {
        launch_variant<MODE, false, false>(st, g, b, a);
    } else if constexpr (MODE == kModeDuplex) {
        if (a.save && a.offs) launch_variant<MODE, true, true>(st, g, b, a);
        else if (a.save) launch_variant<MODE, true, false>(st, g, b, a);
        else if (a.offs) launch_variant<MODE, false, true>(st, g, b, a);
        else launch_variant<MODE, false, false>(st, g, b, a);
    } else {
        if (a.offs) launch_variant<MODE, false, true>(st, g, b, a);
        else launch_variant<MODE, false, false>(st, g, b, a);
    }
}

void launch_composite_duplex(hipStream_t st, const CompositeArgs& a) { launch_mode<kModeDuplex>(st, a); }
void launch_composite_alpha(hipStream_t st, const CompositeArgs& a) { launch_mode<kModeAlpha>(st, a); }
void launch_composite_lcwsr(hipStream_t st, const CompositeArgs& a) { launch_mode<kModeLcwsr>(st, a); }

}  // namespace dgs
