// Training loss of eq. `loss` without its perceptual term,
//     L = (1 - lam) mean |x - y| + lam (1 - mean SSIM(x, y)),
// and dL/dx, for planar [C][H][W] binary32 images (lam = lambda_1 = 0.2 in
// the paper's experimental settings).  SSIM per channel from an 11 x 11
// Gaussian window (sigma 1.5, weights summing to 1), the image zero outside
// its borders, c1 = 0.01^2, c2 = 0.03^2.
//
// Two passes, each streaming down strips of 64 columns: a wavefront (a
// workgroup of its own) owns one strip (lane l: column c0 + l) and a number of
// output rows (strip_rows); it walks those rows and the 5 above and below
// them top to bottom, loading each row (with the 5-column halo on either
// side) a few rows ahead, blurs it along the row from an LDS row buffer, and
// keeps the last 11 row sums in registers for the blur along the column -- no
// workgroup barriers, no 2D tile in LDS:
//   k_ssim_fwd  window statistics of x and y -> the SSIM map; per-strip sums
//               of SSIM and |x - y| (binary64) and, when a gradient is
//               wanted, the three per-pixel coefficients of dL/dx:
//               dL/d mu_x, dL/d E[x^2], dL/d E[xy];
//   k_ssim_bwd  dL/dx = blur(dL/d mu_x) + 2 x blur(dL/d E[x^2])
//               + y blur(dL/d E[xy]) + (1 - lam)/n sign(x - y)
//               (the window is symmetric, so the adjoint of the zero-filled
//               blur is the same blur);
//   loss_sum    the strip sums in a fixed order -> L (binary64, stored as
//               binary32): the result does not depend on scheduling.  One more
//               workgroup of the backward pass; a launch of its own (k_loss_sum)
//               without one.
// The rows are unrolled by 11, the period of the register rings (unrolled
// whole, 42 rows were more code than the instruction cache holds).  The
// forward is bound by its VALU work (235 instructions a row, of them 110
// multiply-adds and 33 products for the sums; keeping the products in the row
// buffer instead took 61 us for 54), the backward by memory (five planes read, one
// written): 3 x 1600 x 1200 54 and 42 us, 71 and 49 before; 3 x 843 x 178,
// whose 32-row strips left most SIMDs idle, 16 and 13 us, 35 and 26 before.
#include <math.h>

#include <string>

#include "ctx.h"

using namespace dgs;

namespace {

constexpr int kTaps = 11, kRad = 5;
constexpr int kStrip = 64;                      // columns per wavefront (one per lane)
constexpr int kAhead = 4;                       // input rows loaded ahead
constexpr int kRowBuf = kStrip + 2 * kRad + 6;  // one row and its halo (+ padding)
constexpr int kSimds = 1024;                    // of 256 CUs
constexpr float kC1 = 0.01f * 0.01f, kC2 = 0.03f * 0.03f;

struct Window {
    float g[kTaps];
};

struct LossArgs {
    const float* x;
    const float* y;
    int C, H, W;
    int rows;        // output rows of a strip: 11 k + 1
    int nx, ny;      // strips along a row, along a column
    float dls;       // dL/dSSIM at every pixel: -lam / n
    float l1c;       // (1 - lam) / n
    float* coef;     // [3][C][H][W], null: loss only
    double* part;    // [strips][2]: sum of SSIM, sum of |x - y|
    float* grad;     // [C][H][W]
    double n, lam;   // pixels, lambda
    float* loss;
};

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Orders a wavefront's LDS row-buffer writes before its reads (and the
// reads before the next row's writes): the lanes exchange values through it.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A strip's columns: lane l reads column c0 - 5 + l, lanes below 10 also
// column c0 + 59 + l (the right halo); zero outside the image.
struct StripCols {
    int ca, cb;
    bool hb;
    __device__ __forceinline__ StripCols(int c0, int lane)
        : ca(c0 - kRad + lane), cb(c0 + kStrip - kRad + lane), hb(lane < 2 * kRad) {}
    __device__ __forceinline__ void load(const float* P, int H, int W, int gy, float& va, float& vb) const {
        const bool rin = gy >= 0 && gy < H;
        const size_t row = (size_t)(rin ? gy : 0) * W;
        va = rin && ca >= 0 && ca < W ? P[row + ca] : 0.0f;
        vb = rin && hb && cb < W ? P[row + cb] : 0.0f;
    }
};

// The strip of a workgroup: neighbours share input rows and columns, and the
// backward reads the coefficients that the forward wrote, so each XCD has one
// contiguous range of them in both.
struct Strip {
    int c, c0, r0;
    __device__ __forceinline__ Strip(const LossArgs& a, int t)
        : c(t / (a.nx * a.ny)), c0(t % a.nx * kStrip), r0(t / a.nx % a.ny * a.rows) {}
};

// L from one wavefront's sums of the strips' (lane i: strips i, i + 64, ... in
// that order).
__device__ __forceinline__ void store_loss(const LossArgs& a, double s, double l, int lane) {
    s = wave_sum(s);
    l = wave_sum(l);
    if (lane == 0) *a.loss = (float)((1.0 - a.lam) * l / a.n + a.lam * (1.0 - s / a.n));
}

// The strip sums by one wavefront, then L: beside the strips of the backward.
__device__ void loss_sum(const LossArgs& a, int strips, int lane) {
    double s = 0.0, l = 0.0;
    const double2* part = reinterpret_cast<const double2*>(a.part);
#pragma unroll 8
    for (int t = lane; t < strips; t += 64) {
        const double2 p = part[t];
        s += p.x;
        l += p.y;
    }
    store_loss(a, s, l, lane);
}

// a / b from i = 1 / b: the product corrected by its remainder.
__device__ __forceinline__ float quotient(float a, float b, float i) {
    const float q = a * i;
    return fmaf(fmaf(-q, b, a), i, q);
}

template <bool GRAD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_ssim_fwd(LossArgs a, Window w) {
    __shared__ float bx[kRowBuf], by[kRowBuf];
    const int lane = threadIdx.x;
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    const Strip st(a, t);
    const size_t plane = (size_t)a.H * a.W, n = (size_t)a.C * plane;
    const float* X = a.x + st.c * plane;
    const float* Y = a.y + st.c * plane;
    const StripCols cols(st.c0, lane);
    const int gx = st.c0 + lane;
    // indexed by input row modulo 11; of the loads kAhead rows are live, of the centres 6
    float ax[kTaps], hx[kTaps], ay[kTaps], hy[kTaps], cx[kTaps], cy[kTaps];
    float ring[kTaps][5];  // row sums of x, y, x^2, y^2, xy of the last 11 rows
    double ssum = 0.0, l1sum = 0.0;
#pragma unroll
    for (int i = 0; i < kAhead; i++) {
        cols.load(X, a.H, a.W, st.r0 - kRad + i, ax[i], hx[i]);
        cols.load(Y, a.H, a.W, st.r0 - kRad + i, ay[i], hy[i]);
    }
    const int rin = min(a.rows, a.H - st.r0) + 2 * kRad;  // input rows that count
    for (int base = 0; base < rin; base += kTaps) {
#pragma unroll
        for (int j = 0; j < kTaps; j++) {
            // input row base + j: image row r0 - 5 + base + j
            const int jl = (j + kAhead) % kTaps, gl = st.r0 - kRad + base + j + kAhead;
            wave_sync();  // the previous row's reads are done
            bx[lane] = ax[j];
            by[lane] = ay[j];
            if (cols.hb) {
                bx[kStrip + lane] = hx[j];
                by[kStrip + lane] = hy[j];
            }
            wave_sync();
            cols.load(X, a.H, a.W, gl, ax[jl], hx[jl]);
            cols.load(Y, a.H, a.W, gl, ay[jl], hy[jl]);
            float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f, s4 = 0.0f;
#pragma unroll
            for (int k = 0; k < kTaps; k++) {
                const float xv = bx[lane + k], yv = by[lane + k], g = w.g[k];
                s0 = fmaf(g, xv, s0);
                s1 = fmaf(g, yv, s1);
                s2 = fmaf(g, xv * xv, s2);
                s3 = fmaf(g, yv * yv, s3);
                s4 = fmaf(g, xv * yv, s4);
            }
            ring[j][0] = s0;
            ring[j][1] = s1;
            ring[j][2] = s2;
            ring[j][3] = s3;
            ring[j][4] = s4;
            cx[j] = bx[lane + kRad];
            cy[j] = by[lane + kRad];
            const int i = base + j;
            if (i < 2 * kRad || i >= rin) continue;
            // output row r0 + i - 10, whose centre is input row i - 5
            const int gy = st.r0 + i - 2 * kRad;
            if (gx >= a.W) continue;
            float m[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < kTaps; k++) {
                const float g = w.g[k];
#pragma unroll
                for (int q = 0; q < 5; q++) m[q] = fmaf(g, ring[(j + 1 + k) % kTaps][q], m[q]);
            }
            const float mx = m[0], my = m[1];
            const float sxx = m[2] - mx * mx, syy = m[3] - my * my, sxy = m[4] - mx * my;
            const float a1 = 2.0f * mx * my + kC1, a2 = 2.0f * sxy + kC2;
            const float b1 = mx * mx + my * my + kC1, b2 = sxx + syy + kC2;
            const float sv = (a1 * a2) / (b1 * b2);
            const int jc = (j + kTaps - kRad) % kTaps;
            ssum += (double)sv;
            l1sum += (double)fabsf(cx[jc] - cy[jc]);
            if (GRAD) {
                // S = a1 a2 / (b1 b2): d/d mu_x through a1 (2 mu_y), a2 (-2 mu_y),
                // b1 (2 mu_x), b2 (-2 mu_x); d/d E[x^2] through b2; d/d E[xy] through a2
                // (with a2 from S cancelled against the division by a2, so that
                // only b1, b2 >= c1, c2 are divided by).  Where x is near y the terms
                // cancel, and what is left of the larger 1 / b2 must be exact: a
                // quotient of equal numbers is 1, S the product of the two, and
                // no product is fused with the sum of it and its negative.
#pragma clang fp contract(off)
                const float i1 = 1.0f / b1, i2 = 1.0f / b2;
                const float q1 = quotient(a1, b1, i1), q2 = quotient(a2, b2, i2), s = q1 * q2;
                const size_t p = st.c * plane + (size_t)gy * a.W + gx;
                a.coef[p] = 2.0f * a.dls * (i1 * (my * q2 - mx * s) - i2 * (my * q1 - mx * s));
                a.coef[n + p] = -(a.dls * s) * i2;
                a.coef[2 * n + p] = 2.0f * (a.dls * q1 * i2);
            }
        }
    }
    ssum = wave_sum(ssum);
    l1sum = wave_sum(l1sum);
    if (lane == 0) {
        a.part[2 * (size_t)t] = ssum;
        a.part[2 * (size_t)t + 1] = l1sum;
    }
}

// Workgroup 0 sums the loss, the others take the strips.
__global__ __launch_bounds__(64) void k_ssim_bwd(LossArgs a, Window w) {
    __shared__ float rb[3][kRowBuf];
    const int lane = threadIdx.x;
    if (blockIdx.x == 0) {
        loss_sum(a, (int)gridDim.x - 1, lane);
        return;
    }
    // shifted by the block of the sum, so that a strip's XCD is the forward's
    const int strips = (int)gridDim.x - 1, b = (int)blockIdx.x < strips ? (int)blockIdx.x : 0;
    const Strip st(a, xcd_remap(b, strips));
    const size_t plane = (size_t)a.H * a.W, n = (size_t)a.C * plane;
    const float* X = a.x + st.c * plane;
    const float* Y = a.y + st.c * plane;
    const float* cf[3] = {a.coef + st.c * plane, a.coef + n + st.c * plane, a.coef + 2 * n + st.c * plane};
    const StripCols cols(st.c0, lane);
    const int gx = st.c0 + lane;
    float av[kTaps][3], hv[kTaps][3];  // indexed by input row modulo 11; kAhead rows live
    float xr[kTaps], yr[kTaps];        // x, y of the output row, by its last input row
    float ring[kTaps][3];              // row sums of the three coefficient planes of the last 11 rows
#pragma unroll
    for (int i = 0; i < kAhead; i++)
#pragma unroll
        for (int q = 0; q < 3; q++) cols.load(cf[q], a.H, a.W, st.r0 - kRad + i, av[i][q], hv[i][q]);
    const int rin = min(a.rows, a.H - st.r0) + 2 * kRad;
    for (int base = 0; base < rin; base += kTaps) {
#pragma unroll
        for (int j = 0; j < kTaps; j++) {
            const int i = base + j, jl = (j + kAhead) % kTaps;
            wave_sync();
#pragma unroll
            for (int q = 0; q < 3; q++) {
                rb[q][lane] = av[j][q];
                if (cols.hb) rb[q][kStrip + lane] = hv[j][q];
            }
            wave_sync();
#pragma unroll
            for (int q = 0; q < 3; q++)
                cols.load(cf[q], a.H, a.W, st.r0 - kRad + i + kAhead, av[jl][q], hv[jl][q]);
            {
                const int gl = st.r0 + i + kAhead - 2 * kRad;
                const bool in = gl >= st.r0 && gl < a.H && gx < a.W;
                const size_t p = (size_t)(in ? gl : 0) * a.W + (in ? gx : 0);
                xr[jl] = X[p];
                yr[jl] = Y[p];
            }
            float s[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < kTaps; k++) {
                const float g = w.g[k];
#pragma unroll
                for (int q = 0; q < 3; q++) s[q] = fmaf(g, rb[q][lane + k], s[q]);
            }
#pragma unroll
            for (int q = 0; q < 3; q++) ring[j][q] = s[q];
            if (i < 2 * kRad || i >= rin || gx >= a.W) continue;
            float m[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < kTaps; k++) {
                const float g = w.g[k];
#pragma unroll
                for (int q = 0; q < 3; q++) m[q] = fmaf(g, ring[(j + 1 + k) % kTaps][q], m[q]);
            }
            const float xv = xr[j], yv = yr[j];
            const float sg = (float)(xv > yv) - (float)(xv < yv);
            a.grad[st.c * plane + (size_t)(st.r0 + i - 2 * kRad) * a.W + gx] =
                fmaf(a.l1c, sg, fmaf(yv, m[2], fmaf(2.0f * xv, m[1], m[0])));
        }
    }
}

// The same sums, in the same order, where nothing runs beside them: 16 wavefronts
// bring the strips' sums to LDS, 4096 at a time.  (One wavefront with
// eight loads in flight took 3 us more for 3 x 1920 x 1080.)
constexpr int kSumThreads = 1024, kSumItems = 4;
__global__ __launch_bounds__(kSumThreads) void k_loss_sum(LossArgs a, int strips) {
    __shared__ double2 buf[kSumThreads * kSumItems];
    const int tid = threadIdx.x;
    const double2* part = reinterpret_cast<const double2*>(a.part);
    double s = 0.0, l = 0.0;
    for (int t0 = 0; t0 < strips; t0 += kSumThreads * kSumItems) {
        const int n = min(strips - t0, kSumThreads * kSumItems);
        double2 p[kSumItems];
#pragma unroll
        for (int i = 0; i < kSumItems; i++) p[i] = part[t0 + min(tid + i * kSumThreads, n - 1)];
#pragma unroll
        for (int i = 0; i < kSumItems; i++) buf[tid + i * kSumThreads] = p[i];
        __syncthreads();
        if (tid < 64)
#pragma unroll 4
            for (int t = tid; t < n; t += 64) {
                s += buf[t].x;
                l += buf[t].y;
            }
        __syncthreads();  // buf is written again
    }
    if (tid < 64) store_loss(a, s, l, tid);
}

// Output rows of a strip, 11 k + 1 (with the 10 rows of its window a whole
// number of ring periods): the least (strips per SIMD + 2) x (rows + 10).  A
// row takes a wavefront about as long alone as two more strips on its SIMD
// add: 3 x 1600 x 1200 with its gradient takes 80, 87, 89 and 119 us in 23,
// 34, 45 and 67 rows, 4, 3, 2 and 2 strips per SIMD.  Of equal ones the most
// rows, which read least: 3 x 1920 x 1080 in 12 and 34 rows (cost 220 both) 98 and
// 86 us with the gradient, 55 and 44 without; 3 x 2560 x 1440 in 23 and 45 140 and
// 133.
int strip_rows(int64_t columns, int H) {
    int best = 12;
    double least = INFINITY;
    for (int rows = 12; rows <= 67; rows += kTaps) {
        const int64_t strips = columns * ((H + rows - 1) / rows), per = (strips + kSimds - 1) / kSimds;
        const double cost = (double)(per + 2) * (rows + 2 * kRad);
        if (cost <= least) {
            least = cost;
            best = rows;
        }
    }
    return best;
}

// The 11 window weights: exp(-t^2 / (2 sigma^2)) for t = -5..5, divided by
// their sum (binary64, then rounded).
Window make_window() {
    double g[kTaps], sum = 0.0;
    for (int i = 0; i < kTaps; i++) {
        const double t = (double)(i - kRad) / 1.5;
        g[i] = exp(-0.5 * t * t);
        sum += g[i];
    }
    Window w;
    for (int i = 0; i < kTaps; i++) w.g[i] = (float)(g[i] / sum);
    return w;
}

template <class T>
hipError_t ensure_buf(T*& p, int64_t& cap, int64_t want, hipStream_t st) {
    if (want <= cap && p) return hipSuccess;
    if (p) {
        hipStreamSynchronize(st);
        hipFree(p);
        p = nullptr;
        cap = 0;
    }
    const hipError_t e = hipMalloc((void**)&p, sizeof(T) * (size_t)want);
    if (e == hipSuccess) cap = want;
    return e;
}

}  // namespace

extern "C" {

dgs_status dgs_loss_l1_ssim(dgs_ctx c, const float* image, const float* target, int32_t channels, int32_t height,
                            int32_t width, float lambda, float* loss, float* grad_image) {
    if (!c) return DGS_ERR_INVALID_ARG;
    if (channels < 1 || channels > 65535 || height < 1 || height > 32767 || width < 1 || width > 32767) {
        c->err = "loss: channels must be in 1..65535, height and width in 1..32767";
        return DGS_ERR_INVALID_ARG;
    }
    if (!(lambda >= 0.0f && lambda <= 1.0f)) {
        c->err = "loss: lambda must be in [0, 1]";
        return DGS_ERR_INVALID_ARG;
    }
    if (!image || !target || !loss) {
        c->err = "loss: NULL image, target or loss pointer";
        return DGS_ERR_INVALID_ARG;
    }
    hipSetDevice(c->device);
    const int64_t n = (int64_t)channels * height * width;
    LossArgs a;
    a.nx = (width + kStrip - 1) / kStrip;
    a.rows = strip_rows((int64_t)a.nx * channels, height);
    a.ny = (height + a.rows - 1) / a.rows;
    const int64_t strips = (int64_t)a.nx * a.ny * channels;
    hipError_t e = ensure_buf(c->loss_part, c->cap_loss_part, 2 * strips, c->stream);
    if (e == hipSuccess && grad_image) e = ensure_buf(c->loss_coef, c->cap_loss_coef, 3 * n, c->stream);
    if (e != hipSuccess) {
        c->err = std::string("loss: hipMalloc failed: ") + hipGetErrorString(e);
        return DGS_ERR_OOM;
    }
    a.x = image;
    a.y = target;
    a.C = channels;
    a.H = height;
    a.W = width;
    a.dls = (float)(-(double)lambda / (double)n);
    a.l1c = (float)((1.0 - (double)lambda) / (double)n);
    a.coef = c->loss_coef;
    a.part = c->loss_part;
    a.grad = grad_image;
    a.n = (double)n;
    a.lam = (double)lambda;
    a.loss = loss;
    const Window w = make_window();
    const dim3 grid((unsigned)strips), block(64);
    if (grad_image) {
        hipLaunchKernelGGL(k_ssim_fwd<true>, grid, block, 0, c->stream, a, w);
        hipLaunchKernelGGL(k_ssim_bwd, dim3((unsigned)strips + 1), block, 0, c->stream, a, w);
    } else {
        hipLaunchKernelGGL(k_ssim_fwd<false>, grid, block, 0, c->stream, a, w);
        hipLaunchKernelGGL(k_loss_sum, dim3(1), dim3(kSumThreads), 0, c->stream, a, (int)strips);
    }
    e = hipGetLastError();
    if (e != hipSuccess) {
        c->err = std::string("loss: kernel launch failed: ") + hipGetErrorString(e);
        return DGS_ERR_DEVICE;
    }
    return DGS_OK;
}

}  // extern "C"
