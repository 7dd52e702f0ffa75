// Neural decode of cells (Sec. III-A neural Gaussians; Sec. IV-A cell
// proxy): each cell's K Gaussians come from its latent feature f_n, the
// viewing distance delta_n and direction d_n through four two-layer MLPs
// F_sigma (tanh), F_c (sigmoid), F_s (sigmoid scale ratio) and F_q (raw
// quaternion); centres follow eq. scaffold_offset with the offsets in the
// cell frame, mu = x_n + R(Q_n)(O^pos * S_n), and scales eqs. nerual_scales
// and scale_res, s = max(0, min(sigmoid(y_s), 1 - |O^pos|)) * S_n.
//
// Mapping: one decoder per workgroup (blockIdx.y), one cell per thread.  The
// workgroup copies its decoder's weights to LDS (at most 51 KB) and every lane
// reads them from there as broadcasts, four to a ds_read_b128, which four
// multiply-adds then use: the second layer's are stored output-major,
// so that both layers read four consecutive ones.  (Read through the scalar
// cache, the four decoders' weights missed its 16 KB and every wavefront
// waited on the L2.)  The second layer's outputs pass through LDS from one
// cell per lane to one Gaussian per lane: the attributes and offsets of
// consecutive Gaussians are consecutive, and a lane per cell touched a line of
// its own with every 4-byte store, K times over.
// Bound by latency (the copies of weights and features, the exchanges through
// LDS) and by the LDS reads, twice the multiply-adds' issue time: 67 us for the
// 83,000 visible cells of the 1920 x 1080 orbit at F = H = 32, K = 10 (121
// through the scalar cache and a lane per cell throughout), 38 us for 20,000
// cells at F = 48, H = 64, K = 4 (290, its registers spilled).  Two cells per
// thread halve the LDS reads but leave too few wavefronts: 96 and 50 us.
// CH, the hidden units held in registers, is 32 or 64.  The opacity decoder,
// whose second layer is the smallest, also places the centres.
//
// The scales, quaternions and centres decide each Gaussian's pixel box, so
// they are computed in binary32 in one fixed order: every sum is a chain of
// fused multiply-adds in ascending index order starting from the bias, the
// sigmoid uses the exp below, and no other contraction happens.  Opacity and
// colour only enter the continuous layer.
#include "common.h"
#include "launch.h"

namespace dgs {

constexpr int kDecodeWaves = 4, kDecodeThreads = 64 * kDecodeWaves;
constexpr int kDecodeSlots = 20;          // outputs per cell of the LDS buffer, at most
constexpr size_t kVoteLds = 256;                     // of __syncthreads_or
constexpr size_t kDecodeLds = 64 * 1024 - kVoteLds;  // dynamic LDS: 64 KB in all, at most

// Orders a wavefront's own LDS accesses: its lanes exchange values through it.
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// exp(x) in binary32: Cody-Waite reduction x = n ln2 + r with ln2 split so
// that n * ln2_hi is exact, the degree-7 Taylor polynomial of e^r in Horner
// form, then the exact scaling by 2^n; one rounding per operation.
__device__ inline float exp32_def(float x) {
#pragma clang fp contract(off)
    x = fminf(88.0f, fmaxf(-88.0f, x));
    const float log2e = 1.44269504088896341f;
    const float ln2_hi = 0.693145751953125f, ln2_lo = 1.42860682030941723e-6f;
    const float n = rintf(x * log2e);
    const float r = (x - n * ln2_hi) - n * ln2_lo;
    float p = 1.0f / 5040.0f;
    p = p * r + 1.0f / 720.0f;
    p = p * r + 1.0f / 120.0f;
    p = p * r + 1.0f / 24.0f;
    p = p * r + 1.0f / 6.0f;
    p = p * r + 0.5f;
    p = p * r + 1.0f;
    p = p * r + 1.0f;
    return ldexpf(p, (int)n);
}

__device__ inline float sigmoid32_def(float y) {
#pragma clang fp contract(off)
    return 1.0f / (1.0f + exp32_def(-y));
}

// Rotation of a cell quaternion (w, x, y, z), normalised first.
__device__ inline void cell_rot32(float w, float x, float y, float z, float* R) {
#pragma clang fp contract(off)
    const float n = sqrtf(((w * w + x * x) + y * y) + z * z);
    w = w / n; x = x / n; y = y / n; z = z / n;
    const float xx = x * x, yy = y * y, zz = z * z;
    const float xy = x * y, xz = x * z, yz = y * z;
    const float wx = w * x, wy = w * y, wz = w * z;
    R[0] = 1.0f - 2.0f * (yy + zz); R[1] = 2.0f * (xy - wz);        R[2] = 2.0f * (xz + wy);
    R[3] = 2.0f * (xy + wz);        R[4] = 1.0f - 2.0f * (xx + zz); R[5] = 2.0f * (yz - wx);
    R[6] = 2.0f * (xz - wy);        R[7] = 2.0f * (yz + wx);        R[8] = 1.0f - 2.0f * (xx + yy);
}

// A decoder's weights in LDS: W1 [I][CH], b1 [CH], W2 [O][CH] output-major, b2
// [O].  Hidden units beyond H have zero weights in and -0 out: their product
// -0 leaves any sum as it is.
struct DecoderLds {
    float *w1, *b1, *w2, *b2;
};

__host__ __device__ inline size_t decode_lds_floats(int I, int CH, int O) { return (size_t)I * CH + CH + (size_t)O * CH + O; }

// Members of a cell per round through the LDS buffer of `slots` outputs per
// cell: the rounds are even, and a lane's row of the buffer has an odd length.
__device__ __forceinline__ int members_per_round(int K, int A, int slots) {
    const int most = ((slots / A) - 1) | 1;
    const int rounds = (K + most - 1) / most;
    return (K + rounds - 1) / rounds;
}

// The wavefront's 64 cells from n0 on, one per lane (live: the ones to decode).
// buf: its buffer, 64 x slots outputs.
template <int CH, int A>
__device__ inline void decode_cells(const DecodeArgs& a, const DecoderLds& w, float* buf, int slots, int n0, uint64_t live,
                                    int lane) {
#pragma clang fp contract(off)
    const int N = a.N, K = a.K, F = a.F;
    const CamK& k = a.fr->k;
    const int64_t M = (int64_t)N * K;
    const int m = (live >> lane) & 1 ? n0 + lane : 0;  // the lane's cell, or cell 0 in its place
    const float ex = a.cell_pos[m] - k.o[0], ey = a.cell_pos[(int64_t)N + m] - k.o[1];
    const float ez = a.cell_pos[2 * (int64_t)N + m] - k.o[2];
    const float dist = sqrtf((ex * ex + ey * ey) + ez * ez);
    // layer 1, input by input: h_j = b1_j + x_0 W1_0j + x_1 W1_1j + ...
    float h[CH];
#pragma unroll
    for (int j = 0; j < CH; j++) h[j] = w.b1[j];
    const auto input = [&](int i, float x) __attribute__((always_inline)) {
        const float4* row = reinterpret_cast<const float4*>(w.w1 + i * CH);
#pragma unroll
        for (int j = 0; j < CH / 4; j++) {
            const float4 q = row[j];
            h[4 * j] = fmaf(x, q.x, h[4 * j]);
            h[4 * j + 1] = fmaf(x, q.y, h[4 * j + 1]);
            h[4 * j + 2] = fmaf(x, q.z, h[4 * j + 2]);
            h[4 * j + 3] = fmaf(x, q.w, h[4 * j + 3]);
        }
    };
    // eight features at a time, the next eight in flight meanwhile
    constexpr int kBlock = 8;
    float x[kBlock];
#pragma unroll
    for (int q = 0; q < kBlock; q++) x[q] = a.features[(int64_t)min(q, F - 1) * N + m];
    for (int i0 = 0; i0 < F; i0 += kBlock) {
        float nx[kBlock];
#pragma unroll
        for (int q = 0; q < kBlock; q++) nx[q] = a.features[(int64_t)min(i0 + kBlock + q, F - 1) * N + m];
#pragma unroll
        for (int q = 0; q < kBlock; q++)
            if (i0 + q < F) input(i0 + q, x[q]);  // uniform
#pragma unroll
        for (int q = 0; q < kBlock; q++) x[q] = nx[q];
    }
    input(F, dist);
    input(F + 1, ex / dist);
    input(F + 2, ey / dist);
    input(F + 3, ez / dist);
#pragma unroll
    for (int j = 0; j < CH; j++) h[j] = h[j] > 0.0f ? h[j] : 0.0f;
    const int G = members_per_round(K, A, slots), row = G | 1, plane = 64 * row;
    const bool color = A == 3 && blockIdx.y == 1;
    for (int k0 = 0; k0 < K; k0 += G) {
        const int gc = min(G, K - k0);
        // layer 2 of members k0 .. k0 + gc - 1, a cell per lane:
        // y_o = b2_o + h_0 W2_0o + h_1 W2_1o + ...
        for (int kk = 0; kk < gc; kk++) {
            float y[A];
#pragma unroll
            for (int o = 0; o < A; o++) y[o] = w.b2[(k0 + kk) * A + o];
            const float* w2 = w.w2 + (size_t)(k0 + kk) * A * CH;
#pragma unroll
            for (int j = 0; j < CH / 4; j++) {
                float4 q[A];
#pragma unroll
                for (int o = 0; o < A; o++) q[o] = reinterpret_cast<const float4*>(w2 + o * CH)[j];
#pragma unroll
                for (int o = 0; o < A; o++) {
                    y[o] = fmaf(h[4 * j], q[o].x, y[o]);
                    y[o] = fmaf(h[4 * j + 1], q[o].y, y[o]);
                    y[o] = fmaf(h[4 * j + 2], q[o].z, y[o]);
                    y[o] = fmaf(h[4 * j + 3], q[o].w, y[o]);
                }
            }
#pragma unroll
            for (int o = 0; o < A; o++) buf[o * plane + lane * row + kk] = y[o];
        }
        wave_order();
        // a Gaussian per lane (e / gc through a float: e < 2^12, exact as
        // (e + 0.5) / gc is at least 0.5 / gc off any integer)
        const float inv = 1.0f / (float)gc;
        for (int e = lane; e < 64 * gc; e += 64) {
            const int cell = (int)(((float)e + 0.5f) * inv), kk = e - cell * gc;
            if (!((live >> cell) & 1)) continue;
            const int n = n0 + cell;
            const int64_t g = (int64_t)n * K + k0 + kk;
            const float* yb = buf + cell * row + kk;
            if constexpr (A == 1) {
                a.opac[g] = tanhf(yb[0]);
                // centre in the cell frame
                float R[9];
                cell_rot32(a.cell_rot[n], a.cell_rot[(int64_t)N + n], a.cell_rot[2 * (int64_t)N + n],
                           a.cell_rot[3 * (int64_t)N + n], R);
                const float u0 = a.offsets[g] * a.cell_scale[n], u1 = a.offsets[M + g] * a.cell_scale[(int64_t)N + n],
                            u2 = a.offsets[2 * M + g] * a.cell_scale[2 * (int64_t)N + n];
                a.means[g] = a.cell_pos[n] + ((R[0] * u0 + R[1] * u1) + R[2] * u2);
                a.means[M + g] = a.cell_pos[(int64_t)N + n] + ((R[3] * u0 + R[4] * u1) + R[5] * u2);
                a.means[2 * M + g] = a.cell_pos[2 * (int64_t)N + n] + ((R[6] * u0 + R[7] * u1) + R[8] * u2);
            } else if constexpr (A == 4) {
#pragma unroll
                for (int o = 0; o < 4; o++) a.rots[o * M + g] = yb[o * plane];
            } else if (color) {
#pragma unroll
                for (int o = 0; o < 3; o++) a.color[o * M + g] = 1.0f / (1.0f + __expf(-yb[o * plane]));
            } else {
                const float o0 = a.offsets[g], o1 = a.offsets[M + g], o2 = a.offsets[2 * M + g];
                const float lim = 1.0f - sqrtf((o0 * o0 + o1 * o1) + o2 * o2);
#pragma unroll
                for (int o = 0; o < 3; o++) {
                    float r = sigmoid32_def(yb[o * plane]);
                    r = r < lim ? r : lim;
                    r = r > 0.0f ? r : 0.0f;
                    a.scales[o * M + g] = r * a.cell_scale[(int64_t)o * N + n];
                }
            }
        }
        wave_order();  // the buffer is reused by the next round
    }
}

template <int CH>
__global__ __launch_bounds__(kDecodeThreads) __attribute__((amdgpu_waves_per_eu(CH == 32 ? 4 : 2))) void k_decode(DecodeArgs a, int slots) {
    extern __shared__ float s_w[];
    const int dec = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int A = dec == 0 ? 1 : dec == 3 ? 4 : 3;  // outputs per Gaussian of this decoder
    const int H = a.H, I = a.F + 4, O = a.K * A;
    // the cells, before the weights: a workgroup with none visible has no work
    const int n0 = (int)(blockIdx.x * kDecodeWaves + wave) * 64, n = n0 + lane;
    const uint64_t live = __ballot(n < a.N && (a.cell_ntiles == nullptr || a.cell_ntiles[n] != 0));
    if (!__syncthreads_or(live != 0)) return;
    DecoderLds w;
    w.w1 = s_w;
    w.w2 = w.w1 + I * CH;  // 16-byte aligned: CH is a multiple of four
    w.b1 = w.w2 + (size_t)O * CH;
    w.b2 = w.b1 + CH;
    float* buf = w.b2 + O + (size_t)wave * 64 * slots;
    const float* W1 = a.weights + a.woff[dec];
    const float* b1 = W1 + (int64_t)I * H;
    const float* W2 = b1 + H;
    const float* b2 = W2 + (int64_t)H * O;
    // several loads in flight per thread: one at a time, a copy of 4,000 weights
    // takes 20 us
#pragma unroll 8
    for (int q = tid; q < I * CH; q += kDecodeThreads) {
        const int i = q / CH, j = q % CH;
        w.w1[q] = j < H ? W1[(int64_t)i * H + j] : 0.0f;
    }
    for (int j = tid; j < CH; j += kDecodeThreads) w.b1[j] = j < H ? b1[j] : 0.0f;
    for (int o = lane; o < O; o += 64)
#pragma unroll 8
        for (int j = wave; j < CH; j += kDecodeWaves) w.w2[o * CH + j] = j < H ? W2[(int64_t)j * O + o] : -0.0f;
    for (int o = tid; o < O; o += kDecodeThreads) w.b2[o] = b2[o];
    __syncthreads();
    if (!live) return;  // uniform per wavefront
    if (dec == 0) decode_cells<CH, 1>(a, w, buf, slots, n0, live, lane);
    else if (dec == 3) decode_cells<CH, 4>(a, w, buf, slots, n0, live, lane);
    else decode_cells<CH, 3>(a, w, buf, slots, n0, live, lane);
}

template <int CH>
static void decode(hipStream_t st, const DecodeArgs& a) {
    const size_t weights = decode_lds_floats(a.F + 4, CH, 4 * a.K) * sizeof(float);
    const size_t per_slot = kDecodeThreads * sizeof(float);
    // outputs per cell in the LDS buffer: at least the four of one quaternion
    int slots = (int)((kDecodeLds - weights) / per_slot);
    slots = slots < kDecodeSlots ? slots : kDecodeSlots;
    hipLaunchKernelGGL(k_decode<CH>, dim3((unsigned)((a.N + kDecodeThreads - 1) / kDecodeThreads), 4), dim3(kDecodeThreads),
                       weights + slots * per_slot, st, a, slots);
}

void launch_decode(hipStream_t st, const DecodeArgs& a) {
    if (a.N <= 0) return;
    if (a.H <= 32) decode<32>(st, a);
    else decode<64>(st, a);
}

}  // namespace dgs
