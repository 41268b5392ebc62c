// Surrogate network for the near-surface integrals: a 216 -> 128 -> 128 -> 4
// MLP with tanh-approximated GELU, input the 6 x 6 x 6 window of phi / h
// around a core data point (offsets -2..3, x fastest), output
// (K_W, h K_grad).  Training (forward, backward, Adam) and inference run on
// BF16 MFMA (v_mfma_f32_16x16x32_bf16) with FP32 accumulation; the first
// layer splits its input into BF16 hi and lo parts (x = hi + lo, two MFMAs)
// so the input keeps about 16 significant bits.
//
// MFMA lane layout used throughout (16 x 16 x 32, wave64, lane l, r = l % 16,
// q = l / 16):  A[m][k] with m = r, k = 8q + j (j = 0..7);
//               B[k][n] with k = 8q + j, n = r;
//               C[m][n] with m = 4q + i (i = 0..3), n = r.
// A wavefront owns a tile of 16 samples; activations move from the C layout
// to the A layout of the next layer through a row-major BF16 tile in LDS.
//
// Parameters are FP32 masters in one packed vector (W1[128][216], b1[128],
// W2[128][128], b2[128], W3[4][128], b3[4]), with BF16 copies laid out for
// the B operands: W1 [128][224] (zero padded), W2 [128][128], its transpose
// for the backward pass, W3 [16][128] (rows 4..15 zero).
#include <float.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "fraction.hpp"
#include "window.hpp"

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kIn = 216, kInPad = 224, kH = 128, kOut = 4;
constexpr int kNParam = 44804;
constexpr int oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kOut * kH;
static_assert(oB3 + kOut == kNParam, "parameter layout");

struct MlpDev {
    const float *w;      // FP32 masters
    const bf16 *w1b;     // [128][224]
    const bf16 *w2b;     // [128][128]
    const bf16 *w2tb;    // [128][128], transposed
    const bf16 *w3b;     // [16][128]
};

__device__ __forceinline__ floatx4 mfma(const bf16x8 &a, const bf16x8 &b, const floatx4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 ld8(const bf16 *p) { return *reinterpret_cast<const bf16x8 *>(p); }

// GELU in its tanh form, 0.5 z (1 + tanh(u)) with u = sqrt(2/pi) (z + 0.044715
// z^3), evaluated as z s with s = 0.5 (1 + tanh(u)) = 1 / (1 + exp(-2u)): the
// same function.  exp(-2u) = 2^(k z (1 + 0.044715 z^2)) with k = -2 sqrt(2/pi)
// / ln 2 folded into the polynomial, on the hardware's base-2 exponential and
// reciprocal (each within one ulp; the activations dominate the network's
// vector work, and an IEEE division would cost ten instructions more).  For
// large |u| the exponential saturates to 0 or inf and s to 1 or 0.
__device__ __forceinline__ float gelu_s(float z) {
    const float a = z * __builtin_fmaf(-0.1029432395800235f, z * z, -2.302208198144325f);
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(a));
}

__device__ __forceinline__ float gelu(float z) { return z * gelu_s(z); }

// d/dz [z s] = s + z s (1 - s) 2 u'(z), u' = sqrt(2/pi) (1 + 3 * 0.044715 z^2)
// (the tanh form's 0.5 (1 + th) + 0.5 z (1 - th^2) u' with th = 2s - 1).
__device__ __forceinline__ float gelu_grad(float z) {
    const float s = gelu_s(z);
    return s + 2.0f * z * s * (1.0f - s) * 0.7978845608028654f * (1.0f + 3.0f * 0.044715f * z * z);
}

struct Tile {
    floatx4 z1[8], z2[8];
    floatx4 y;
};

// Forward pass of one 16-sample tile.  `xs(m, k0, v)` returns the 8 inputs
// k0..k0+7 of sample m (zero past 215).  `a1`, `a2` are the wave's row-major
// [16][128] BF16 activation tiles in LDS.  Ends with the wave's LDS writes
// complete; callers synchronise the workgroup between phases.
template <class XSrc>
__device__ __forceinline__ void forward_tile(const XSrc &xs, const MlpDev &W, bf16 *a1, bf16 *a2, Tile &T, int lane) {
    const int r = lane & 15, q = lane >> 4;
    // every accumulator starts from its bias (the column's hidden unit)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float bb = W.w[oB1 + 16 * t + r];
        T.z1[t] = floatx4{bb, bb, bb, bb};
    }
    for (int s = 0; s < kInPad / 32; ++s) {
        float v[8];
        xs(r, 32 * s + 8 * q, v);
        bf16x8 ah, al;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bf16 hi = (bf16)v[j];
            ah[j] = hi;
            al[j] = (bf16)(v[j] - (float)hi);
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const bf16x8 b = ld8(W.w1b + (16 * t + r) * kInPad + 32 * s + 8 * q);
            T.z1[t] = mfma(ah, b, T.z1[t]);
            T.z1[t] = mfma(al, b, T.z1[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) a1[(4 * q + i) * kH + 16 * t + r] = (bf16)gelu(T.z1[t][i]);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float bb = W.w[oB2 + 16 * t + r];
        T.z2[t] = floatx4{bb, bb, bb, bb};
    }
#pragma unroll
    for (int s = 0; s < kH / 32; ++s) {
        const bf16x8 a = ld8(a1 + r * kH + 32 * s + 8 * q);
#pragma unroll
        for (int t = 0; t < 8; ++t) T.z2[t] = mfma(a, ld8(W.w2b + (16 * t + r) * kH + 32 * s + 8 * q), T.z2[t]);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) a2[(4 * q + i) * kH + 16 * t + r] = (bf16)gelu(T.z2[t][i]);
    __syncthreads();
    const float b3 = r < kOut ? W.w[oB3 + r] : 0.f;
    T.y = floatx4{b3, b3, b3, b3};
#pragma unroll
    for (int s = 0; s < kH / 32; ++s)
        T.y = mfma(ld8(a2 + r * kH + 32 * s + 8 * q), ld8(W.w3b + r * kH + 32 * s + 8 * q), T.y);
}

struct GlobalX {
    const float *x;
    int64_t base, B;
    __device__ __forceinline__ void operator()(int m, int k0, float *v) const {
        const int64_t s = base + m;
        if (s < B && k0 + 8 <= kIn) {
            const float4 a = *reinterpret_cast<const float4 *>(x + s * kIn + k0);
            const float4 b = *reinterpret_cast<const float4 *>(x + s * kIn + k0 + 4);
            v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
            v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = 0.f;
        }
    }
};

// ---------------------------------------------------------------------------
// Training, in three kernels.  A batch of a few thousand samples is little
// work (0.3 GFLOP a step at 2048), so its time is latency: how many dependent
// memory and LDS round trips follow each other, and over how many CUs the
// work is spread.
//   train_rows_kernel   forward and backward of 16 samples per workgroup;
//   weight_grad_kernel  the weight gradients, a product over the samples,
//                       split over output tiles and over chunks of samples;
//   reduce_kernel       sum of the chunks in a fixed order and the Adam step.
// One kernel with 64 samples per workgroup for the first two (32 workgroups
// at 2048 samples) took 65 us, then 9 us for the sum, 5 us for Adam and 4 us
// for a copy of the loss; these three take 10, 9 and 5 us.
//
// The first kernel hands its activations and errors to the second as BF16
// rows of samples, one row per unit: [a1 128 | a2 128 | d1 128 | d2 128 |
// dy 4][Bp], Bp = B rounded up to kTrainChunk (rows past B carry no error).
// The C layout holds four consecutive samples of a unit per lane, so these
// rows are written in 8-byte pieces, and the operands of the products over
// the samples are 16-byte pieces of them.  dY is handed on in FP32 too (the
// output biases' gradient), with each workgroup's loss.
//
// Sums go in a fixed order: the samples of a chunk, then the chunks one by one.
// Up to kMaxChunks chunks of kTrainChunk samples that is the order of a running
// sum over partial gradients of 64 samples; a change in it would be an ulp in
// the gradient, but Adam divides by the gradient's own size, and 16 steps later
// a batch in ten has its outputs 1e-4 apart.
// ---------------------------------------------------------------------------
constexpr int kTrainRows = 16;         // samples per workgroup of the first kernel
constexpr int kTrainChunk = 64;        // samples per chunk: two MFMA steps, at least
constexpr int kMaxChunks = 256;        // partial gradients kept (46 MB)
constexpr int kActUnits = 4 * kH + kOut;
constexpr int rA1 = 0, rA2 = kH, rD1 = 2 * kH, rD2 = 3 * kH, rDY = 4 * kH;
constexpr int kActPad = kH + 8;        // LDS row of activations, padded by 16 bytes (banks)

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Forward and backward of 16 samples: four wavefronts, each the hidden units
// 32 w .. 32 w + 31 of every layer (two column tiles), so the chain of one
// layer is a quarter of a wavefront's that takes all 128.  All weights and
// inputs are requested at the start.  Every value is computed in the order of
// forward_tile.
__global__ __launch_bounds__(256, 1) void train_rows_kernel(MlpDev W, const float *__restrict__ x, int64_t B,
                                                            const float *__restrict__ t_in,
                                                            const float *__restrict__ dy_in, float4 lw,
                                                            bf16 *__restrict__ acts, int64_t Bp,
                                                            float *__restrict__ dys, float *__restrict__ tile_loss) {
    __shared__ __attribute__((aligned(16))) bf16 s_a1[kTrainRows * kActPad];
    __shared__ __attribute__((aligned(16))) bf16 s_a2[kTrainRows * kActPad];
    __shared__ __attribute__((aligned(16))) bf16 s_d2[kTrainRows * kActPad];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
    const int64_t base = (int64_t)blockIdx.x * kTrainRows;
    constexpr int S1 = kInPad / 32, S2 = kH / 32;
    const int n0 = 32 * w + r, n1 = n0 + 16;   // this lane's hidden units
    float4 xa[S1], xb[S1];
    {
        const bool in = base + r < B;
        const float *row = x + (in ? base + r : 0) * kIn;
#pragma unroll
        for (int s = 0; s < S1; ++s) {
            const int k0 = 32 * s + 8 * q;
            const float *p = row + (k0 < kIn ? k0 : 0);
            xa[s] = *reinterpret_cast<const float4 *>(p);
            xb[s] = *reinterpret_cast<const float4 *>(p + 4);
            if (!in || k0 >= kIn) xa[s] = xb[s] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
    bf16x8 w1[2][S1], w2[2][S2], w2t[2][S2], w3[S2];
#pragma unroll
    for (int s = 0; s < S1; ++s) {
        w1[0][s] = ld8(W.w1b + n0 * kInPad + 32 * s + 8 * q);
        w1[1][s] = ld8(W.w1b + n1 * kInPad + 32 * s + 8 * q);
    }
#pragma unroll
    for (int s = 0; s < S2; ++s) {
        w2[0][s] = ld8(W.w2b + n0 * kH + 32 * s + 8 * q);
        w2[1][s] = ld8(W.w2b + n1 * kH + 32 * s + 8 * q);
        w2t[0][s] = ld8(W.w2tb + n0 * kH + 32 * s + 8 * q);
        w2t[1][s] = ld8(W.w2tb + n1 * kH + 32 * s + 8 * q);
        w3[s] = ld8(W.w3b + r * kH + 32 * s + 8 * q);
    }
    const float b1[2] = {W.w[oB1 + n0], W.w[oB1 + n1]}, b2[2] = {W.w[oB2 + n0], W.w[oB2 + n1]};
    const float b3 = r < kOut ? W.w[oB3 + r] : 0.f;
    float w3f[2][kOut];
#pragma unroll
    for (int o = 0; o < kOut; ++o) {
        w3f[0][o] = W.w[oW3 + o * kH + n0];
        w3f[1][o] = W.w[oW3 + o * kH + n1];
    }
    float dy[4], lsum = 0.f;   // targets, then errors, of the samples 4q .. 4q + 3, output r
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t m = base + 4 * q + i;
        dy[i] = r < kOut && m < B ? (dy_in ? dy_in : t_in)[m * kOut + r] : 0.f;
    }

    floatx4 z1[2], z2[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        z1[c] = floatx4{b1[c], b1[c], b1[c], b1[c]};
        z2[c] = floatx4{b2[c], b2[c], b2[c], b2[c]};
    }
#pragma unroll
    for (int s = 0; s < S1; ++s) {
        const float v[8] = {xa[s].x, xa[s].y, xa[s].z, xa[s].w, xb[s].x, xb[s].y, xb[s].z, xb[s].w};
        bf16x8 ah, al;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bf16 hi = (bf16)v[j];
            ah[j] = hi;
            al[j] = (bf16)(v[j] - (float)hi);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            z1[c] = mfma(ah, w1[c][s], z1[c]);
            z1[c] = mfma(al, w1[c][s], z1[c]);
        }
    }
    // four consecutive samples of one unit: to the unit's row, and (for the
    // next layer's A operand) to the samples' rows in LDS
    auto hand_on = [&](const float (&v)[4], int unit, int row0, bf16 *lds) {
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[i] = (bf16)v[i];
            if (lds) lds[(4 * q + i) * kActPad + unit] = o[i];
        }
        *reinterpret_cast<bf16x4 *>(acts + (int64_t)(row0 + unit) * Bp + base + 4 * q) = o;
    };
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float g[4] = {gelu(z1[c][0]), gelu(z1[c][1]), gelu(z1[c][2]), gelu(z1[c][3])};
        hand_on(g, c ? n1 : n0, rA1, s_a1);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < S2; ++s) {
        const bf16x8 a = ld8(s_a1 + r * kActPad + 32 * s + 8 * q);
#pragma unroll
        for (int c = 0; c < 2; ++c) z2[c] = mfma(a, w2[c][s], z2[c]);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float g[4] = {gelu(z2[c][0]), gelu(z2[c][1]), gelu(z2[c][2]), gelu(z2[c][3])};
        hand_on(g, c ? n1 : n0, rA2, s_a2);
    }
    __syncthreads();
    // every wavefront takes the output layer, so that each has dY
    floatx4 y = floatx4{b3, b3, b3, b3};
#pragma unroll
    for (int s = 0; s < S2; ++s) y = mfma(ld8(s_a2 + r * kActPad + 32 * s + 8 * q), w3[s], y);
    if (dy_in == nullptr) {
        const float wo = r == 0 ? lw.x : (r == 1 ? lw.y : (r == 2 ? lw.z : lw.w));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float e = y[i] - dy[i];
            const bool in = r < kOut && base + 4 * q + i < B;   // rows past B contribute nothing
            lsum = in ? fmaf(wo * e, e, lsum) : lsum;
            dy[i] = in ? 2.0f * wo * e / (float)B : 0.f;
        }
    }
    if (w == 0) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) lsum += __shfl_down(lsum, off);
        if (lane == 0) tile_loss[blockIdx.x] = lsum;
        if (r < kOut) {
            hand_on(dy, r, rDY, nullptr);
            *reinterpret_cast<float4 *>(dys + r * Bp + base + 4 * q) = make_float4(dy[0], dy[1], dy[2], dy[3]);
        }
    }
    // dA2 = dY W3 (K = 4, FP32 masters), dZ2 = dA2 * gelu'(z2)
    {
        float d[2][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float d0 = __shfl(dy[i], 16 * q), d1 = __shfl(dy[i], 16 * q + 1), d2 = __shfl(dy[i], 16 * q + 2),
                        d3 = __shfl(dy[i], 16 * q + 3);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float da = d0 * w3f[c][0] + d1 * w3f[c][1] + d2 * w3f[c][2] + d3 * w3f[c][3];
                d[c][i] = da * gelu_grad(z2[c][i]);
            }
        }
        hand_on(d[0], n0, rD2, s_d2);
        hand_on(d[1], n1, rD2, s_d2);
    }
    __syncthreads();
    // dA1 = dZ2 W2 (B operand from the transposed copy), dZ1 = dA1 * gelu'(z1)
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < S2; ++s) {
        const bf16x8 a = ld8(s_d2 + r * kActPad + 32 * s + 8 * q);
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[c] = mfma(a, w2t[c][s], acc[c]);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        float d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = acc[c][i] * gelu_grad(z1[c][i]);
        hand_on(d, c ? n1 : n0, rD1, nullptr);
    }
}

// Weight gradients C[o][i] = sum over a chunk's samples of D[m][o] S[m][i].
// One wavefront per column tile of 16 inputs i and chunk: it reads its B
// operand once and the eight A operands of all 128 outputs (roles 0..13: W1,
// whose inputs are x rounded to BF16; 14..21: W2; 22: W3, one A and eight B
// operands).  Role 23 takes the biases, the errors' sums over the samples in
// their order, one row of errors per lane.
constexpr int kRolesW1 = kInPad / 16, kRolesW2 = kH / 16, kRoles = kRolesW1 + kRolesW2 + 2;
static_assert(kRoles % 4 == 0, "four roles per workgroup");

__device__ __forceinline__ void bias_grad(const bf16 *acts, const float *dys, int64_t Bp, int64_t first, int units,
                                          float *P, int lane) {
#pragma unroll 1
    for (int h = 0; h < kH / 64; ++h) {
        const int o = 64 * h + lane;
        const bf16 *d1 = acts + (int64_t)(rD1 + o) * Bp + first, *d2 = acts + (int64_t)(rD2 + o) * Bp + first;
        float s1 = 0.f, s2 = 0.f;
        for (int u = 0; u < units; ++u) {
            bf16x8 a[kTrainChunk / 8], b[kTrainChunk / 8];
#pragma unroll
            for (int k = 0; k < kTrainChunk / 8; ++k) {
                a[k] = ld8(d1 + kTrainChunk * u + 8 * k);
                b[k] = ld8(d2 + kTrainChunk * u + 8 * k);
            }
            float t1 = 0.f, t2 = 0.f;
#pragma unroll
            for (int m = 0; m < kTrainChunk; ++m) {
                t1 += (float)a[m / 8][m % 8];
                t2 += (float)b[m / 8][m % 8];
            }
            s1 += t1;
            s2 += t2;
        }
        P[oB1 + o] = s1;
        P[oB2 + o] = s2;
    }
    if (lane < kOut) {
        float s3 = 0.f;
        for (int u = 0; u < units; ++u) {
            float4 v[kTrainChunk / 4];
#pragma unroll
            for (int k = 0; k < kTrainChunk / 4; ++k)
                v[k] = *reinterpret_cast<const float4 *>(dys + lane * Bp + first + kTrainChunk * u + 4 * k);
            float t = 0.f;
#pragma unroll
            for (int k = 0; k < kTrainChunk / 4; ++k) t = (((t + v[k].x) + v[k].y) + v[k].z) + v[k].w;
            s3 += t;
        }
        P[oB3 + lane] = s3;
    }
}

__global__ __launch_bounds__(256) void weight_grad_kernel(const float *__restrict__ x, int64_t B,
                                                          const bf16 *__restrict__ acts,
                                                          const float *__restrict__ dys, int64_t Bp, int steps,
                                                          float *__restrict__ part) {
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int role = (int)(blockIdx.x % (kRoles / 4)) * 4 + (threadIdx.x >> 6);
    const int64_t chunk = blockIdx.x / (kRoles / 4);
    const int64_t first = chunk * steps * 32;
    float *P = part + chunk * kNParam;
    if (role == kRoles - 1) {
        const int64_t left = (Bp - first) / kTrainChunk, mine = steps * 32 / kTrainChunk;
        bias_grad(acts, dys, Bp, first, (int)(left < mine ? left : mine), P, lane);
        return;
    }
    floatx4 acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 zero;
#pragma unroll
    for (int j = 0; j < 8; ++j) zero[j] = (bf16)0.f;
    const bool is_w1 = role < kRolesW1, is_w2 = !is_w1 && role < kRolesW1 + kRolesW2, is_w3 = role == kRolesW1 + kRolesW2;
    const int it = is_w1 ? role : role - kRolesW1;
    const int col = 16 * it + r;
    const bf16 *rows8 = acts + (int64_t)((is_w1 ? rD1 : (is_w3 ? rA2 : rD2)) + r) * Bp;   // eight tiles' operands
    const bf16 *row1 = acts + (int64_t)(is_w3 ? rDY + (r < kOut ? r : 0) : rA1 + (is_w2 ? col : 0)) * Bp;
    for (int s = 0; s < steps; ++s) {
        const int64_t m0 = first + 32 * s + 8 * q;
        if (first + 32 * s >= Bp) break;   // the same for the whole wavefront
        bf16x8 one;
        if (is_w1) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t m = m0 + j < B ? m0 + j : B - 1;   // rows past B meet d1 = 0
                v[j] = x[m * kIn + (col < kIn ? col : 0)];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) one[j] = (bf16)(m0 + j < B && col < kIn ? v[j] : 0.f);
        } else {
            one = ld8(row1 + m0);
            if (is_w3 && r >= kOut) one = zero;
        }
        bf16x8 many[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) many[t] = ld8(rows8 + (int64_t)(16 * t) * Bp + m0);
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = is_w3 ? mfma(one, many[t], acc[t]) : mfma(many[t], one, acc[t]);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int o = 16 * t + 4 * q + j;   // output (W1, W2)
            if (is_w1) {
                if (col < kIn) P[oW1 + o * kIn + col] = acc[t][j];
            } else if (is_w2) {
                P[oW2 + o * kH + col] = acc[t][j];
            } else if (4 * q + j < kOut) {
                P[oW3 + (4 * q + j) * kH + 16 * t + r] = acc[t][j];
            }
        }
}

// Refresh the BF16 operand copies of parameter p from the FP32 master.
__device__ __forceinline__ void write_bf16_copy(int p, float v, bf16 *w1b, bf16 *w2b, bf16 *w2tb, bf16 *w3b) {
    if (p < oB1) {
        const int o = p / kIn, i = p % kIn;
        w1b[o * kInPad + i] = (bf16)v;
    } else if (p >= oW2 && p < oB2) {
        const int o = (p - oW2) / kH, i = (p - oW2) % kH;
        w2b[o * kH + i] = (bf16)v;
        w2tb[i * kH + o] = (bf16)v;
    } else if (p >= oW3 && p < oB3) {
        const int o = (p - oW3) / kH, i = (p - oW3) % kH;
        w3b[o * kH + i] = (bf16)v;
    }
}

__global__ __launch_bounds__(256) void sync_copies_kernel(const float *__restrict__ w, bf16 *w1b, bf16 *w2b,
                                                          bf16 *w2tb, bf16 *w3b) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < kNParam) write_bf16_copy(p, w[p], w1b, w2b, w2tb, w3b);
}

struct AdamArgs {
    float *w, *m, *v;
    float lr, b1, b2, eps, c1, c2;
    bf16 *w1b, *w2b, *w2tb, *w3b;
};

// Adam (Kingma & Ba 2015) with bias correction, then the BF16 copies.
__device__ __forceinline__ void adam_update(const AdamArgs &A, int p, float gp) {
    const float mp = A.b1 * A.m[p] + (1.0f - A.b1) * gp;
    const float vp = A.b2 * A.v[p] + (1.0f - A.b2) * gp * gp;
    A.m[p] = mp;
    A.v[p] = vp;
    const float wp = A.w[p] - A.lr * (mp / A.c1) / (sqrtf(vp / A.c2) + A.eps);
    A.w[p] = wp;
    write_bf16_copy(p, wp, A.w1b, A.w2b, A.w2tb, A.w3b);
}

__global__ __launch_bounds__(256) void adam_kernel(AdamArgs A, const float *__restrict__ g) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < kNParam) adam_update(A, p, g[p]);
}

// Gradient of parameter p = sum over the chunks of part[c][p], in chunk order
// (deterministic); written to `grad`, or given to Adam at once.  The last
// workgroup sums the loss, four tiles (64 samples) at a time, in their order.
constexpr int kReduceBlocks = (kNParam + 255) / 256 + 1;

template <bool ADAM>
__global__ __launch_bounds__(256) void reduce_kernel(const float *__restrict__ part, int n_part,
                                                     const float *__restrict__ tile_loss, int64_t n_tiles,
                                                     float *__restrict__ grad, AdamArgs A,
                                                     float *__restrict__ loss_out) {
    if (blockIdx.x == kReduceBlocks - 1) {
        __shared__ float s[256];
        if (loss_out == nullptr) return;
        const int64_t units = n_tiles / 4;
        float sum = 0.f;
        for (int64_t u0 = 0; u0 < units; u0 += 256) {
            const int64_t u = u0 + threadIdx.x;
            if (u < units) {
                const float4 t = reinterpret_cast<const float4 *>(tile_loss)[u];
                s[threadIdx.x] = ((t.x + t.y) + t.z) + t.w;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                const int n = (int)(units - u0 < 256 ? units - u0 : 256);
#pragma unroll 8
                for (int k = 0; k < n; ++k) sum += s[k];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss_out = sum;
        return;
    }
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= kNParam) return;
    float s = 0.f;
#pragma unroll 8
    for (int g = 0; g < n_part; ++g) s += part[(int64_t)g * kNParam + p];
    if (ADAM)
        adam_update(A, p, s);
    else
        grad[p] = s;
}

// Forward only, for [B][216] inputs.
__global__ __launch_bounds__(256) void forward_kernel(MlpDev W, const float *__restrict__ x, int64_t B,
                                                      float *__restrict__ y) {
    __shared__ __attribute__((aligned(16))) bf16 s_a1[64 * kH];
    __shared__ __attribute__((aligned(16))) bf16 s_a2[64 * kH];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
    const int64_t base = (int64_t)blockIdx.x * 64 + 16 * w;
    Tile T;
    forward_tile(GlobalX{x, base, B}, W, s_a1 + 16 * w * kH, s_a2 + 16 * w * kH, T, lane);
    if (r < kOut)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t s = base + 4 * q + i;
            if (s < B) y[s * kOut + r] = T.y[i];
        }
}

}  // namespace

// ---------------------------------------------------------------------------
// Handle
// ---------------------------------------------------------------------------
struct sgrid_mlp {
    int device = 0;
    float *w = nullptr, *m = nullptr, *v = nullptr;
    bf16 *w1b = nullptr, *w2b = nullptr, *w2tb = nullptr, *w3b = nullptr;
    // training workspace: partial gradients [chunk][parameter], dY by rows and
    // the tiles' losses, and the rows of activations and errors, for up to
    // train_rows samples
    float *part = nullptr, *dys = nullptr, *tile_loss = nullptr;
    bf16 *acts = nullptr;
    int64_t train_rows = 0;
    int64_t step = 0;
    float gate_tau = FLT_MAX;     // non-planarity threshold (mean squared residual, units of h^2)
    float kw_lo = -0.05f, kw_hi = 1.05f;
    uint32_t *fallback = nullptr;  // fallback cell list of the learned integrals
    int64_t fallback_cap = 0;
    // Calls that use the model are ordered across streams: each records `done`
    // on its stream, and a call on another stream first waits for it.
    hipEvent_t done = nullptr;
    hipStream_t last = nullptr;
    bool used = false;
    MlpDev dev() const { return MlpDev{w, w1b, w2b, w2tb, w3b}; }
};

namespace sgrid {

static void free_mlp(sgrid_mlp *m) {
    if (!m) return;
    void *ptrs[] = {m->w, m->m, m->v, m->w1b, m->w2b, m->w2tb, m->w3b, m->part, m->dys, m->tile_loss, m->acts, m->fallback};
    for (void *p : ptrs) dev_free(p);
    if (m->done) (void)hipEventDestroy(m->done);
    delete m;
}

// Start of a call that uses the model's buffers on stream `st`: wait for the
// model's previous call when that ran on another stream.
static sgrid_status begin_use(const sgrid_mlp *mc, hipStream_t st) {
    sgrid_mlp *m = const_cast<sgrid_mlp *>(mc);
    if (m->used && m->last != st) SG_CHECK_HIP(hipStreamWaitEvent(st, m->done, 0));
    return SGRID_OK;
}

// End of such a call: later calls on other streams wait for this point.
static sgrid_status end_use(const sgrid_mlp *mc, hipStream_t st) {
    sgrid_mlp *m = const_cast<sgrid_mlp *>(mc);
    SG_CHECK_HIP(hipEventRecord(m->done, st));
    m->last = st;
    m->used = true;
    return SGRID_OK;
}

// How a batch is split: rounded up to whole chunks of kTrainChunk samples, at
// most kMaxChunks of them (then longer ones).
struct TrainSplit {
    int64_t rows, tiles;
    int chunks, steps;
    explicit TrainSplit(int64_t B) {
        const int64_t units = (B + kTrainChunk - 1) / kTrainChunk;
        const int64_t per = (units + kMaxChunks - 1) / kMaxChunks;
        rows = units * kTrainChunk;
        tiles = rows / kTrainRows;
        chunks = (int)((units + per - 1) / per);
        steps = (int)(per * (kTrainChunk / 32));
    }
};

// The training workspace for t, and the fallback list below: growing a buffer frees
// the old block, which kernels queued by earlier calls (on any stream) may still use,
// so the device is waited for before it goes back to the allocator, which may give it
// to the next request of that size.
static sgrid_status ensure_train(sgrid_mlp *m, const TrainSplit &t) {
    if (t.rows <= m->train_rows) return SGRID_OK;
    if (m->part || m->dys || m->tile_loss || m->acts) SG_CHECK_HIP(hipDeviceSynchronize());
    dev_free(m->part);
    dev_free(m->dys);
    dev_free(m->tile_loss);
    dev_free(m->acts);
    m->part = m->dys = m->tile_loss = nullptr;
    m->acts = nullptr;
    m->train_rows = 0;
    const int64_t chunks = std::min<int64_t>(t.rows / kTrainChunk, kMaxChunks);
    sgrid_status s = dev_alloc((void **)&m->part, (size_t)chunks * kNParam * 4, "MLP partial gradients");
    if (s != SGRID_OK) return s;
    s = dev_alloc((void **)&m->dys, (size_t)t.rows * kOut * 4, "MLP output errors");
    if (s != SGRID_OK) return s;
    s = dev_alloc((void **)&m->tile_loss, (size_t)t.tiles * 4, "MLP partial losses");
    if (s != SGRID_OK) return s;
    s = dev_alloc((void **)&m->acts, (size_t)t.rows * kActUnits * sizeof(bf16), "MLP activations");
    if (s != SGRID_OK) return s;
    m->train_rows = t.rows;
    return SGRID_OK;
}

sgrid_status mlp_ensure_fallback(sgrid_mlp *m, int64_t cells) {
    if (cells <= m->fallback_cap) return SGRID_OK;
    if (m->fallback) SG_CHECK_HIP(hipDeviceSynchronize());
    dev_free(m->fallback);
    m->fallback = nullptr;
    m->fallback_cap = 0;
    sgrid_status s = dev_alloc((void **)&m->fallback, (size_t)(cells + 1) * 4, "fallback list");
    if (s != SGRID_OK) return s;
    m->fallback_cap = cells;
    return SGRID_OK;
}

// Forward, backward and weight gradients of a batch; the gradient goes to
// `grad` (ADAM false) or into an Adam step (ADAM true).
template <bool ADAM>
static sgrid_status run_backward(sgrid_mlp *m, const float *x, int64_t B, const float *t, const float *dy,
                                 const float lw[4], float *grad, const AdamArgs &A, float *loss, hipStream_t st) {
    const TrainSplit sp(B);
    sgrid_status s = ensure_train(m, sp);
    if (s != SGRID_OK) return s;
    hipLaunchKernelGGL(train_rows_kernel, dim3((unsigned)sp.tiles), dim3(256), 0, st, m->dev(), x, B, t, dy,
                       make_float4(lw[0], lw[1], lw[2], lw[3]), m->acts, sp.rows, m->dys, m->tile_loss);
    SG_CHECK_LAUNCH("MLP forward and backward");
    hipLaunchKernelGGL(weight_grad_kernel, dim3((unsigned)(sp.chunks * (kRoles / 4))), dim3(256), 0, st, x, B, m->acts,
                       m->dys, sp.rows, sp.steps, m->part);
    SG_CHECK_LAUNCH("MLP weight gradient");
    hipLaunchKernelGGL(reduce_kernel<ADAM>, dim3(kReduceBlocks), dim3(256), 0, st, m->part, sp.chunks, m->tile_loss,
                       sp.tiles, grad, A, loss);
    SG_CHECK_LAUNCH("MLP gradient reduction");
    return SGRID_OK;
}

}  // namespace sgrid

extern "C" sgrid_status sgrid_mlp_create(const float *params_host, sgrid_mlp **out) {
    sgrid::clear_error();
    SG_REQUIRE(out != nullptr, "out is NULL");
    *out = nullptr;
    SG_REQUIRE(params_host != nullptr, "params is NULL");
    sgrid_mlp *m = new sgrid_mlp();
    if (hipGetDevice(&m->device) != hipSuccess ||
        hipEventCreateWithFlags(&m->done, hipEventDisableTiming) != hipSuccess) {
        sgrid::set_error("MLP setup: no device or event");
        sgrid::free_mlp(m);
        return SGRID_E_HIP;
    }
    struct A { void **p; size_t bytes; };
    A allocs[] = {{(void **)&m->w, kNParam * 4}, {(void **)&m->m, kNParam * 4}, {(void **)&m->v, kNParam * 4},
                  {(void **)&m->w1b, kH * kInPad * 2}, {(void **)&m->w2b, kH * kH * 2},
                  {(void **)&m->w2tb, kH * kH * 2}, {(void **)&m->w3b, 16 * kH * 2}};
    for (auto &a : allocs) {
        sgrid_status s = sgrid::dev_alloc(a.p, a.bytes, "MLP parameters");
        if (s != SGRID_OK) { sgrid::free_mlp(m); return s; }
    }
    hipError_t e = hipSuccess;
    if (e == hipSuccess) e = hipMemcpy(m->w, params_host, kNParam * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemset(m->m, 0, kNParam * 4);
    if (e == hipSuccess) e = hipMemset(m->v, 0, kNParam * 4);
    if (e == hipSuccess) e = hipMemset(m->w1b, 0, kH * kInPad * 2);
    if (e == hipSuccess) e = hipMemset(m->w3b, 0, 16 * kH * 2);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(sync_copies_kernel, dim3((kNParam + 255) / 256), dim3(256), 0, nullptr, m->w, m->w1b,
                           m->w2b, m->w2tb, m->w3b);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        sgrid::set_error("MLP setup failed: %s", hipGetErrorString(e));
        sgrid::free_mlp(m);
        return SGRID_E_HIP;
    }
    *out = m;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_mlp_destroy(sgrid_mlp *m) {
    sgrid::clear_error();
    if (!m) return SGRID_OK;
    hipError_t e = hipDeviceSynchronize();
    sgrid::free_mlp(m);
    if (e != hipSuccess) {
        sgrid::set_error("hipDeviceSynchronize before destroy failed: %s", hipGetErrorString(e));
        return SGRID_E_HIP;
    }
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_mlp_get_params(const sgrid_mlp *m, float *params_host, float *adam_m_host,
                                             float *adam_v_host, int64_t *step) {
    sgrid::clear_error();
    SG_REQUIRE(m != nullptr, "model is NULL");
    SG_CHECK_HIP(hipDeviceSynchronize());
    if (params_host) SG_CHECK_HIP(hipMemcpy(params_host, m->w, kNParam * 4, hipMemcpyDeviceToHost));
    if (adam_m_host) SG_CHECK_HIP(hipMemcpy(adam_m_host, m->m, kNParam * 4, hipMemcpyDeviceToHost));
    if (adam_v_host) SG_CHECK_HIP(hipMemcpy(adam_v_host, m->v, kNParam * 4, hipMemcpyDeviceToHost));
    if (step) *step = m->step;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_mlp_set_state(sgrid_mlp *m, const float *adam_m_host, const float *adam_v_host,
                                            int64_t step) {
    sgrid::clear_error();
    SG_REQUIRE(m != nullptr && adam_m_host != nullptr && adam_v_host != nullptr, "NULL argument");
    SG_REQUIRE(step >= 0, "step must be >= 0");
    SG_CHECK_HIP(hipDeviceSynchronize());
    SG_CHECK_HIP(hipMemcpy(m->m, adam_m_host, kNParam * 4, hipMemcpyHostToDevice));
    SG_CHECK_HIP(hipMemcpy(m->v, adam_v_host, kNParam * 4, hipMemcpyHostToDevice));
    m->step = step;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_mlp_set_gate(sgrid_mlp *m, float tau, float kw_lo, float kw_hi) {
    sgrid::clear_error();
    SG_REQUIRE(m != nullptr, "model is NULL");
    SG_REQUIRE(tau >= 0.f && kw_lo <= kw_hi, "gate needs tau >= 0 and kw_lo <= kw_hi");
    m->gate_tau = tau;
    m->kw_lo = kw_lo;
    m->kw_hi = kw_hi;
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_mlp_forward(const sgrid_mlp *m, const float *x, int64_t B, float *y, void *stream) {
    sgrid::clear_error();
    SG_REQUIRE(m != nullptr, "model is NULL");
    SG_REQUIRE(B >= 0, "B must be >= 0");
    if (B == 0) return SGRID_OK;
    SG_REQUIRE(x && y && sg_aligned(x, 16) && sg_aligned(y, 16), "x / y NULL or not 16-byte aligned");
    const int64_t nwg = (B + 63) / 64;
    SG_REQUIRE(nwg <= kMaxGrid, "batch too large");
    hipStream_t st = sg_stream(stream);
    sgrid_status s = sgrid::begin_use(m, st);
    if (s != SGRID_OK) return s;
    hipLaunchKernelGGL(forward_kernel, dim3((unsigned)nwg), dim3(256), 0, st, m->dev(), x, B, y);
    SG_CHECK_LAUNCH("MLP forward");
    return sgrid::end_use(m, st);
}

extern "C" sgrid_status sgrid_mlp_backward(sgrid_mlp *m, const float *x, const float *dy, int64_t B, float *grad,
                                           void *stream) {
    sgrid::clear_error();
    SG_REQUIRE(m != nullptr, "model is NULL");
    SG_REQUIRE(B >= 1, "B must be >= 1");
    SG_REQUIRE(x && dy && grad && sg_aligned(x, 16) && sg_aligned(dy, 16) && sg_aligned(grad, 4),
               "x / dy / grad NULL or misaligned");
    SG_REQUIRE((B + 63) / 64 <= kMaxGrid, "batch too large");
    hipStream_t st = sg_stream(stream);
    sgrid_status s = sgrid::begin_use(m, st);
    if (s != SGRID_OK) return s;
    const float lw[4] = {0, 0, 0, 0};
    s = sgrid::run_backward<false>(m, x, B, nullptr, dy, lw, grad, AdamArgs{}, nullptr, st);
    if (s != SGRID_OK) return s;
    return sgrid::end_use(m, st);
}

namespace sgrid {

// The model's next Adam step.  The decay rates are the FP32 numbers nearest
// 0.9 and 0.999, and the bias corrections 1 - beta^t use those same numbers,
// so the step is Adam with these rates.
static AdamArgs next_adam(sgrid_mlp *m, float lr) {
    m->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = (float)(1.0 - pow((double)b1, (double)m->step));
    const float c2 = (float)(1.0 - pow((double)b2, (double)m->step));
    return AdamArgs{m->w, m->m, m->v, lr, b1, b2, 1e-8f, c1, c2, m->w1b, m->w2b, m->w2tb, m->w3b};
}

}  // namespace sgrid

extern "C" sgrid_status sgrid_mlp_train_step(sgrid_mlp *m, const float *x, const float *t, int64_t B,
                                             const float *loss_weights, float lr, float *loss_dev, void *stream) {
    sgrid::clear_error();
    SG_REQUIRE(m != nullptr, "model is NULL");
    SG_REQUIRE(B >= 1, "B must be >= 1");
    SG_REQUIRE(x && t && loss_weights && sg_aligned(x, 16) && sg_aligned(t, 16), "x / t / weights NULL or misaligned");
    SG_REQUIRE(lr >= 0.f, "lr must be >= 0");
    SG_REQUIRE((B + 63) / 64 <= kMaxGrid, "batch too large");
    hipStream_t st = sg_stream(stream);
    sgrid_status s = sgrid::begin_use(m, st);
    if (s != SGRID_OK) return s;
    s = sgrid::ensure_train(m, sgrid::TrainSplit(B));   // before the step counts
    if (s != SGRID_OK) return s;
    s = sgrid::run_backward<true>(m, x, B, t, nullptr, loss_weights, nullptr, sgrid::next_adam(m, lr), loss_dev, st);
    if (s != SGRID_OK) {
        m->step -= 1;
        return s;
    }
    return sgrid::end_use(m, st);
}

extern "C" sgrid_status sgrid_mlp_apply_gradient(sgrid_mlp *m, const float *grad_dev, float lr, void *stream) {
    sgrid::clear_error();
    SG_REQUIRE(m != nullptr, "model is NULL");
    SG_REQUIRE(grad_dev != nullptr && sg_aligned(grad_dev, 4), "grad NULL or misaligned");
    SG_REQUIRE(lr >= 0.f, "lr must be >= 0");
    hipStream_t st = sg_stream(stream);
    sgrid_status s = sgrid::begin_use(m, st);
    if (s != SGRID_OK) return s;
    hipLaunchKernelGGL(adam_kernel, dim3((kNParam + 255) / 256), dim3(256), 0, st, sgrid::next_adam(m, lr), grad_dev);
    SG_CHECK_LAUNCH("Adam");
    return sgrid::end_use(m, st);
}

// ---------------------------------------------------------------------------
// Learned near-surface integrals with gate and plain fallback
// ---------------------------------------------------------------------------
namespace {

using sgrid::kWin;                     // phi window of a package, local -2..6
using sgrid::kWinN;
using sgrid::kVol;
using sgrid::kVolN;

// Stages the 9^3 phi window of core package p into LDS (all threads of the block).
__device__ __forceinline__ void stage_window(const float *__restrict__ phi, const uint32_t *__restrict__ nbr,
                                             int64_t p, float *s_phi, uint32_t *s_ids) {
    if (threadIdx.x < 27) s_ids[threadIdx.x] = nbr[p * 27 + threadIdx.x];
    __syncthreads();
    sgrid::stage_window_part<256>(phi, s_ids, threadIdx.x, s_phi);
    __syncthreads();
}

// Network input of cell c (local index i + 4j + 16k) from the staged window.
struct WindowX {
    const float *f;
    int cell0;
    float inv_h;
    __device__ __forceinline__ void operator()(int m, int k0, float *v) const {
        const int c = cell0 + m;
        const int i = c & 3, j = (c >> 2) & 3, k = c >> 4;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int kk = k0 + e;
            if (kk < kIn) {
                const int ox = kk % 6, oy = (kk / 6) % 6, oz = kk / 36;   // offset + 2
                v[e] = f[(i + ox) + kWin * ((j + oy) + kWin * (k + oz))] * inv_h;
            } else {
                v[e] = 0.f;
            }
        }
    }
};

// Saturation of the cut fraction at the 7^3 tap points: bit 0 = V in {0, 1}
// (fraction_saturated), bit 1 = phi > 0.
__device__ __forceinline__ void saturation_flags(const float *f, float inv_h, float inv_2h, uint8_t *s_sat) {
    for (int v = threadIdx.x; v < kVolN; v += blockDim.x) {
        const int x = v % kVol + 1, y = (v / kVol) % kVol + 1, z = v / (kVol * kVol) + 1;
        const int c = x + kWin * (y + kWin * z);
        const float gx = (f[c + 1] - f[c - 1]) * inv_2h;
        const float gy = (f[c + kWin] - f[c - kWin]) * inv_2h;
        const float gz = (f[c + kWin * kWin] - f[c - kWin * kWin]) * inv_2h;
        const float a = f[c] * inv_h;
        const bool sat = sgrid::fraction_saturated(a, gx, gy, gz);
        s_sat[v] = (uint8_t)((sat ? 1 : 0) | (a > 0.f ? 2 : 0));
    }
}

__global__ __launch_bounds__(256) void zero_u32_kernel(uint32_t *p) { *p = 0u; }
__global__ __launch_bounds__(64) void add_u32_kernel(uint32_t *total, const uint32_t *part) { *total += *part; }

// Learned-integral kernel: two core packages (128 points) per workgroup of
// four wavefronts.
//  1. Each package's 128 lanes stage its 9^3 window, a row per lane, with the
//     BF16 hi + lo parts of the network inputs and the gate's row sums, then
//     the 7^3 tap points' fractions: 1 or 0 where saturated, NaN elsewhere.
//  2. One lane per point sums the 32 taps' fractions.  A point whose taps are
//     all saturated takes that exact sum (the plain value); the others (a
//     NaN) are listed, in LDS, for the network.
//  3. The listed points are spread in 16-point tiles over the wavefronts,
//     tile T on wavefront T mod 4, and each wavefront evaluates the gate of
//     its tiles' points, two lanes per point.
//  4. The network over the tiles: W1's and W2's 32-input slices are staged
//     in LDS once per workgroup (every wavefront takes part in the staging
//     and its barriers) and each weight fragment feeds both of a wavefront's
//     tiles, hi and lo parts.  A wavefront reads back only activation rows it
//     wrote.
//  5. The same wavefront writes the network's value or lists the point for
//     the plain fallback.
// The vector units are busy 65 % of the time, the LDS 60 % (a third of that
// bank conflicts of the gathered inputs), the matrix units 22 %, with the three
// workgroups per CU that registers and LDS allow: 8.3 ms for torus2048's 46 M
// points, 0.60 ms for prism512's 3.6 M.  The same work with 5 % fewer vector
// instructions (an idle wavefront's gate skipped) or with the hidden units
// split over the wavefronts (eleven barriers instead of 23) took as long.
// Every listed point's network row is computed in the MFMA accumulation
// order of forward_tile, so the outputs are the bits of sgrid_mlp_forward on
// the gathered windows.
constexpr int kLearnPkgs = 2;   // packages per workgroup
constexpr int kLearnPts = 64 * kLearnPkgs;
constexpr int kActStride = kH + 8;   // bf16 per activation row in LDS

struct LearnLds {
    float phi[kWinN + 3];
    uint32_t xhl[kWinN + 3];   // BF16 hi (low half) and lo (high half) parts of the window's phi / h
    uint32_t ids[28];
    float v[sgrid::kVWinN];    // V of the saturated tap points (1 or 0), NaN for the others
};

// The gate's sums over one window row for the four positions along x: r0 and
// its x moment.  Kept for the 81 rows of both packages in the activation area
// (past W1's two slices, free until layer 1 ends).
constexpr int kRowSums = 4 * kWin * kWin;

// The weights of layers 1 and 2 pass through LDS, one 32-input slice (128
// rows x 32 BF16, 8 KB) per step, so the workgroup's four wavefronts read each
// slice from L2 once instead of four times.  W1's slices are double-buffered
// in the activation area (free until layer 1 ends); W2's go, one at a time,
// where the windows were (free once every wavefront has evaluated its gate
// and passed layer 1).  Rows are padded to kWRow BF16.
constexpr int kWRow = 40;
constexpr int kWSlice = kH * kWRow;   // BF16 per buffered slice
constexpr int kW1Steps = kInPad / 32, kW2Steps = kH / 32;

// Thread tid's share of slice s of a [128][row_len] weight matrix: row
// tid % 128, inputs 32 s + 16 (tid / 128) .. + 15 (consecutive lanes take
// consecutive rows, 20 words apart in LDS: no bank conflicts).
struct WPart {
    bf16x8 a, b;
};
__device__ __forceinline__ WPart w_load(const bf16 *w, int row_len, int s, int tid) {
    const bf16 *src = w + (tid & 127) * row_len + 32 * s + 16 * (tid >> 7);
    return WPart{ld8(src), ld8(src + 8)};
}
__device__ __forceinline__ void w_store(bf16 *buf, const WPart &v, int tid) {
    bf16 *dst = buf + (tid & 127) * kWRow + 16 * (tid >> 7);
    *reinterpret_cast<bf16x8 *>(dst) = v.a;
    *reinterpret_cast<bf16x8 *>(dst + 8) = v.b;
}

// Activation rows in LDS.  The C layout's four row groups (q) start 4 x 68 =
// 272 words apart, 16 modulo the 32 banks, so rows 8..15 of a tile hold their
// 32-byte column pieces swapped in pairs: the 16 x 16 stores of a column tile
// then cover the banks evenly.  A reader's offset changes by a lane constant.
__device__ __forceinline__ void act_store(bf16 *s_act, int row0, int col, int q, int r, const floatx4 &z) {
    bf16 *dst = s_act + row0 * kActStride + r + (q >> 1 ? col ^ 16 : col);
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef float floatx2 __attribute__((ext_vector_type(2)));
        const floatx2 g = {gelu(z[i]), gelu(z[i + 1])};
        const bf16x2 v = __builtin_convertvector(g, bf16x2);   // one instruction for both
        dst[i * kActStride] = v[0];
        dst[(i + 1) * kActStride] = v[1];
    }
}
// Columns 8 q .. 8 q + 7 of a 32-column slice of row r (modulo 16).
__device__ __forceinline__ int act_piece(int q, int r) { return 8 * (q ^ ((r >> 3) << 1)); }

// The network over the listed points of TILES tiles (rows 16 tile + r of the
// list): layer outputs through the wavefront's own activation rows, the
// outputs y to s_y[row][4].  Every wavefront of the workgroup calls it (TILES
// = 0 for one without tiles: it helps stage the weights and meets the
// barriers), after its gate.
template <int TILES>
__device__ __forceinline__ void learned_network(const MlpDev &W, LearnLds *lds, const int16_t *s_off,
                                                const uint8_t *s_list, int n_list, const int tile[2], bf16 *s_act,
                                                float *s_y, int lane) {
    const int r = lane & 15, q = lane >> 4, tid = threadIdx.x;
    constexpr int NT = TILES > 0 ? TILES : 1;
    int base[NT];
    const LearnLds *win[NT];
#pragma unroll
    for (int m = 0; m < TILES; ++m) {
        const int row = 16 * tile[m] + r;
        const int pt = s_list[row < n_list ? row : n_list - 1];   // rows past the list repeat its last point
        const int c = pt & 63;
        win[m] = lds + (pt >> 6);
        base[m] = (c & 3) + kWin * (((c >> 2) & 3) + kWin * (c >> 4));
    }
    // layer 1: [16 x 224] (hi + lo BF16 parts of phi / h) x W1^T per tile;
    // accumulators start from the biases, as in forward_tile
    floatx4 acc[NT][8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float bb = W.w[oB1 + 16 * t + r];
#pragma unroll
        for (int m = 0; m < TILES; ++m) acc[m][t] = floatx4{bb, bb, bb, bb};
    }
    // slice s + 1 is stored at the start of step s (its buffer was last read in
    // step s - 1, which ended with a barrier) and slice s + 2 loads meanwhile
    WPart part = w_load(W.w1b, kInPad, 0, tid);
    w_store(s_act, part, tid);
    part = w_load(W.w1b, kInPad, 1, tid);
    __syncthreads();
    for (int s = 0; s < kW1Steps; ++s) {
        if (s + 1 < kW1Steps) {
            w_store(s_act + ((s + 1) & 1) * kWSlice, part, tid);
            if (s + 2 < kW1Steps) part = w_load(W.w1b, kInPad, s + 2, tid);
        }
        if (TILES > 0) {
            const bf16 *wb = s_act + (s & 1) * kWSlice;
            bf16x8 bw[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) bw[t] = ld8(wb + (16 * t + r) * kWRow + 8 * q);
#pragma unroll
            for (int m = 0; m < TILES; ++m) {
                bf16x8 ah, al;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int off = base[m] + s_off[32 * s + 8 * q + e];
                    const uint32_t hl = win[m]->xhl[off];   // both parts in one read
                    ah[e] = __builtin_bit_cast(bf16, (uint16_t)(hl & 0xFFFFu));
                    al[e] = __builtin_bit_cast(bf16, (uint16_t)(hl >> 16));
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    acc[m][t] = mfma(ah, bw[t], acc[m][t]);
                    acc[m][t] = mfma(al, bw[t], acc[m][t]);
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int m = 0; m < TILES; ++m) act_store(s_act, 16 * tile[m] + 4 * q, 16 * t, q, r, acc[m][t]);
    // layer 2, W2's slices one at a time in the windows' LDS (a wavefront
    // reads back only activation rows it wrote itself)
    static_assert(sizeof(LearnLds) * kLearnPkgs >= kWSlice * sizeof(bf16), "W2 slice buffer");
    bf16 *w2buf = reinterpret_cast<bf16 *>(lds);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float bb = W.w[oB2 + 16 * t + r];
#pragma unroll
        for (int m = 0; m < TILES; ++m) acc[m][t] = floatx4{bb, bb, bb, bb};
    }
    part = w_load(W.w2b, kH, 0, tid);
    for (int s = 0; s < kW2Steps; ++s) {
        w_store(w2buf, part, tid);
        if (s + 1 < kW2Steps) part = w_load(W.w2b, kH, s + 1, tid);
        __syncthreads();
        if (TILES > 0) {
            bf16x8 bv[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) bv[t] = ld8(w2buf + (16 * t + r) * kWRow + 8 * q);
#pragma unroll
            for (int m = 0; m < TILES; ++m) {
                const bf16x8 a = ld8(s_act + (16 * tile[m] + r) * kActStride + 32 * s + act_piece(q, r));
#pragma unroll
                for (int t = 0; t < 8; ++t) acc[m][t] = mfma(a, bv[t], acc[m][t]);
            }
        }
        __syncthreads();
    }
    if (TILES == 0) return;
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int m = 0; m < TILES; ++m) act_store(s_act, 16 * tile[m] + 4 * q, 16 * t, q, r, acc[m][t]);
    // layer 3
    floatx4 y[NT];
    const float b3 = r < kOut ? W.w[oB3 + r] : 0.f;
#pragma unroll
    for (int m = 0; m < TILES; ++m) y[m] = floatx4{b3, b3, b3, b3};
#pragma unroll
    for (int s = 0; s < kH / 32; ++s) {
        const bf16x8 w3 = ld8(W.w3b + r * kH + 32 * s + 8 * q);
#pragma unroll
        for (int m = 0; m < TILES; ++m)
            y[m] = mfma(ld8(s_act + (16 * tile[m] + r) * kActStride + 32 * s + act_piece(q, r)), w3, y[m]);
    }
    if (r < kOut) {
#pragma unroll
        for (int m = 0; m < TILES; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) s_y[(16 * tile[m] + 4 * q + i) * kOut + r] = y[m][i];
    }
}

__global__ __launch_bounds__(256, 3) void learned_kernel(MlpDev W, const float *__restrict__ phi,
                                                         const uint32_t *__restrict__ nbr,
                                                         const uint32_t *__restrict__ core_list, int64_t n_core,
                                                         int64_t ci0, int64_t ci_end, float inv_h, float inv_2h,
                                                         float tau, float kw_lo, float kw_hi,
                                                         float *__restrict__ out, uint32_t *__restrict__ fb_list,
                                                         uint32_t *__restrict__ fb_count) {
    __shared__ __attribute__((aligned(16))) LearnLds lds[kLearnPkgs];   // 16-byte rows of W2 go here later
    // window offset of network input kk (ox + 9 oy + 81 oz); the padding
    // inputs 216..223 meet zero columns of W1, so they read any finite window
    // value (offset 0) and add exactly zero, without a branch per input
    __shared__ int16_t s_off[kInPad];
    __shared__ __attribute__((aligned(16))) bf16 s_act[kLearnPts * kActStride];   // rows padded by 16 bytes
    __shared__ float s_y[kLearnPts * kOut];
    __shared__ uint8_t s_list[kLearnPts];   // listed points: slot * 64 + local index
    __shared__ uint32_t s_n;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (threadIdx.x < kInPad) {
        const int kk = threadIdx.x;
        s_off[kk] = kk < kIn ? (int16_t)(kk % 6 + kWin * ((kk / 6) % 6) + kWin * kWin * (kk / 36)) : (int16_t)0;
    }
    if (threadIdx.x == 0) s_n = 0u;
    // 1. staging, per package: 128 lanes each
    const int slot = w >> 1, t128 = threadIdx.x & 127;
    LearnLds &L = lds[slot];
    // core packages [ci0, ci_end) of the n_core (outputs are indexed over all)
    const int64_t cw = ci0 + (int64_t)blockIdx.x * kLearnPkgs + slot;
    const bool live = cw < ci_end;                 // a package slot past the end repeats the last package
    const int64_t ci = live ? cw : ci_end - 1;
    const int64_t p = core_list[ci];
    if (t128 < 27) L.ids[t128] = nbr[p * 27 + t128];
    __syncthreads();
    float2 *sums = reinterpret_cast<float2 *>(s_act + 2 * kWSlice);   // [package][row][x position]
    static_assert((2 * kWSlice * sizeof(bf16)) % 8 == 0 &&
                      2 * kWSlice * sizeof(bf16) + kLearnPkgs * kRowSums * sizeof(float2) <=
                          kLearnPts * kActStride * sizeof(bf16),
                  "row sums in the activation area");
    {
        // one window row per lane (81 of a package's 128): phi, the network
        // inputs' hi and lo parts and the gate's row sums from its registers
        sgrid::WindowRows<128> rows(t128);
        rows.load(phi, [&](int s) { return L.ids[s]; });
        float v[kWin];
        rows.values(0, v);
        if (t128 < rows.kRows) {
#pragma unroll
            for (int x = 0; x < kWin; ++x) {
                L.phi[kWin * t128 + x] = v[x];
                const float f = v[x] * inv_h;
                const bf16 hi = (bf16)f;
                const bf16 lo = (bf16)(f - (float)hi);
                L.xhl[kWin * t128 + x] =
                    (uint32_t)__builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const float *u = v + x;
                const float r0 = ((u[0] + u[1]) + (u[2] + u[3])) + (u[4] + u[5]);
                const float rx = fmaf(2.5f, u[5] - u[0], fmaf(1.5f, u[4] - u[1], 0.5f * (u[3] - u[2])));
                sums[slot * kRowSums + 4 * t128 + x] = make_float2(r0, rx);
            }
        }
    }
    __syncthreads();
    {
        // the tap points' saturation, a row of seven per lane and the package's
        // two wavefronts sharing its points
        const int rl = min(lane, kVol * kVol - 1);
        const int ry = rl % kVol, rz = rl / kVol;
        const float *c = L.phi + 1 + kWin * ((ry + 1) + kWin * (rz + 1));
        float *vr = L.v + sgrid::vidx(0, ry - 1, rz - 1);
        auto point = [&](int x) {   // 0..6: window coordinate x - 1
            const float gx = (c[x + 1] - c[x - 1]) * inv_2h;
            const float gy = (c[x + kWin] - c[x - kWin]) * inv_2h;
            const float gz = (c[x + kWin * kWin] - c[x - kWin * kWin]) * inv_2h;
            const float a = c[x] * inv_h;
            const float v = a > 0.f ? 1.f : 0.f;
            vr[(x + 7) & 7] = sgrid::fraction_saturated(a, gx, gy, gz) ? v : __builtin_nanf("");
        };
        if ((w & 1) == 0) {
#pragma unroll
            for (int x = 0; x < 4; ++x) point(x);
        } else {
#pragma unroll
            for (int x = 4; x < kVol; ++x) point(x);
        }
    }
    __syncthreads();
    const int64_t stride = n_core * 64;
    // 2. saturated points: one lane per point (the first 64 of each
    // package's 128) sums its 32 taps' fractions, 1 or 0 by the sign of phi,
    // with the plain kernels' tap sums, so the value is the plain one bit for
    // bit; a point with a cut tap (NaN) is listed
    if (t128 < 64) {
        const int c = t128;
        float kw, kx, ky, kz;
        sgrid::tap_sums([&](int x, int y, int z) { return L.v[sgrid::vidx(x, y, z)]; }, c & 3, (c >> 2) & 3, c >> 4,
                        kw, kx, ky, kz);
        const bool sat = kw == kw;   // a cut tap's NaN reaches the sum
        if (live) {
            if (sat) {
                const int64_t o = ci * 64 + c;
                out[o] = kw;
                out[stride + o] = kx;
                out[2 * stride + o] = ky;
                out[3 * stride + o] = kz;
            } else {
                s_list[atomicAdd(&s_n, 1u)] = (uint8_t)(slot * 64 + c);
            }
        }
    }
    __syncthreads();
    const int n_list = (int)s_n;
    const int n_tiles = (n_list + 15) / 16;
    const int tile[2] = {w, w + 4};
    const int mine = (w < n_tiles ? 1 : 0) + (w + 4 < n_tiles ? 1 : 0);
    if (n_tiles == 0) return;   // the same for the whole workgroup
    // 3. the gate of this wavefront's points, two lanes per point: lanes
    // 0..31 the rows of tile w, lanes 32..63 those of tile w + 4 (before the
    // network, whose second layer reuses the windows' LDS).
    // Non-planarity: mean squared residual of the window after its
    // least-squares affine fit.  The basis 1, ox, oy, oz (offsets centred at
    // 2.5) is orthogonal on the window, so the fit's coefficients are the
    // moments s0 / 216 and s_a / 630.  The residual is then summed over the
    // window a second time, explicitly: the closed form s2 - 216 c0^2 -
    // 630 |c|^2 subtracts nearly equal numbers for the near-planar windows the
    // gate has to tell apart.  An error in the coefficients only moves the sum
    // at second order (the residual is orthogonal to the basis).  Both passes
    // sum phi itself and apply 1/h to the result (for h a power of two the
    // bits of summing phi / h).  Lane `part` takes the window rows 2i + part
    // of the 36 (ez = 2i / 6 for both parities, 6 being even, ey = 2i % 6 +
    // part).
    const int row = 16 * tile[lane >> 5] + ((lane >> 1) & 15), part = lane & 1;
    const bool valid = row < n_list;
    const int pt = s_list[valid ? row : n_list - 1];
    const LearnLds &Lp = lds[pt >> 6];
    const int c = pt & 63;
    const int ci_ = c & 3, cj = (c >> 2) & 3, ck = c >> 4;
    // The first pass takes the rows' sums and x moments from the staging, which
    // has them once per row and x position; each row adds its share to the y
    // and z moments.  Fused and separate operations are written out, so that
    // the decisions do not depend on how the loops are compiled.  A wavefront
    // without points skips both passes.
    const float part_f = (float)part;
    const float ey[3] = {part_f - 2.5f, part_f - 0.5f, part_f + 1.5f};
    const int planes = mine > 0 ? 6 : 0;
    float s0 = 0.f, sx = 0.f, sy = 0.f, sz = 0.f;
    {
        const float2 *rs = sums + (pt >> 6) * kRowSums + 4 * ((cj + part) + kWin * ck) + ci_;
        float ez = -2.5f;
#pragma unroll 2
        for (int z = 0; z < planes; ++z, ez += 1.0f, rs += 4 * kWin) {
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const float2 q = rs[8 * m];
                s0 += q.x;
                sx += q.y;
                sy = fmaf(ey[m], q.x, sy);
                sz = fmaf(ez, q.x, sz);
            }
        }
    }
    s0 += __shfl_xor(s0, 1);
    sx += __shfl_xor(sx, 1);
    sy += __shfl_xor(sy, 1);
    sz += __shfl_xor(sz, 1);
    const float c0 = s0 / 216.f, cx = sx / 630.f, cy = sy / 630.f, cz = sz / 630.f;   // units of phi
    float rr = 0.f;
    {
#pragma clang fp contract(off)
        float px[6], pm[3];
#pragma unroll
        for (int x = 0; x < 6; ++x) px[x] = cx * (x - 2.5f);
#pragma unroll
        for (int m = 0; m < 3; ++m) pm[m] = fmaf(cy, ey[m], c0);
        const float *wrow = Lp.phi + ci_ + kWin * ((cj + part) + kWin * ck);
        float ez = -2.5f;
#pragma unroll 1
        for (int z = 0; z < planes; ++z, ez += 1.0f, wrow += kWin * kWin) {
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                const float pyz = fmaf(cz, ez, pm[m]);
#pragma unroll
                for (int x = 0; x < 6; ++x) {
                    const float e = wrow[2 * kWin * m + x] - (pyz + px[x]);
                    rr = fmaf(e, e, rr);
                }
            }
        }
    }
    rr += __shfl_xor(rr, 1);
    const float res = rr * inv_h * inv_h * (1.0f / 216.f);
    // 4. the network over this wavefront's tiles (every wavefront takes part)
    if (mine == 2)
        learned_network<2>(W, lds, s_off, s_list, n_list, tile, s_act, s_y, lane);
    else if (mine == 1)
        learned_network<1>(W, lds, s_off, s_list, n_list, tile, s_act, s_y, lane);
    else
        learned_network<0>(W, lds, s_off, s_list, n_list, tile, s_act, s_y, lane);
    if (mine == 0) return;
    // 5. the network's value or the fallback list (the point's row and list
    // entry read again rather than kept across the network)
    const int row_o = 16 * tile[lane >> 5] + ((lane >> 1) & 15);
    if (row_o < n_list && (lane & 1) == 0) {
        const int pt_o = s_list[row_o];
        const int64_t o = (ci0 + (int64_t)blockIdx.x * kLearnPkgs + (pt_o >> 6)) * 64 + (pt_o & 63);
        const float *yv = s_y + row_o * kOut;
        if (res <= tau && yv[0] >= kw_lo && yv[0] <= kw_hi) {
            out[o] = yv[0];
            out[stride + o] = yv[1];
            out[2 * stride + o] = yv[2];
            out[3 * stride + o] = yv[3];
        } else {
            fb_list[atomicAdd(fb_count, 1u)] = (uint32_t)o;
        }
    }
}

// Plain integrals of the listed points, `*fb_count` of them, read on the device:
// a persistent grid strides over the list, so its size need not be known at
// launch.  The 32 taps of a point's dual-cell query, each with its own cut
// fraction from central differences, with the plain kernels' fractions and tap
// sums, so the value is the plain one bit for bit.  A wavefront takes kFbPts
// points at a time: one tap per lane, two points per step, kFbStep points' loads
// issued together; the fractions go to LDS, and one lane per point sums them.
// Bound by the latency of its scattered reads (list, core package, neighbour
// row, seven values): 11.6 us for prism512's points and 154 us for torus2048's,
// 35 and 474 us with a lane per point, which took its 32 taps one after another.
constexpr int kFbPts = 16, kFbStep = 8;

__global__ __launch_bounds__(256) void fallback_kernel(const float *__restrict__ phi, const uint32_t *__restrict__ nbr,
                                                       const uint32_t *__restrict__ core_list, int64_t n_core,
                                                       float inv_h, float inv_2h, const uint32_t *__restrict__ fb_list,
                                                       const uint32_t *__restrict__ fb_count, float *__restrict__ out) {
    __shared__ float s_v[4][kFbPts][33];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t count = *fb_count, stride = n_core * 64;
    // this lane's tap: block 0 the eight nearest, 1 to 3 those two cells apart
    // along x, y, z (tap_sums); (tx, ty, tz) relative to the point
    const int half = lane & 32, tap = lane & 31, blk = tap >> 3;
    const int tx = blk == 1 ? 3 * ((tap >> 2) & 1) - 1 : (tap >> 2) & 1;
    const int ty = blk == 2 ? 3 * ((tap >> 1) & 1) - 1 : (tap >> 1) & 1;
    const int tz = blk == 3 ? 3 * (tap & 1) - 1 : tap & 1;
    for (int64_t base = ((int64_t)blockIdx.x * 4 + w) * kFbPts; base < count; base += (int64_t)gridDim.x * 4 * kFbPts) {
        const int n = (int)(count - base < kFbPts ? count - base : kFbPts);
        const int mine = lane % kFbPts;
        const uint32_t o = fb_list[base + (mine < n ? mine : n - 1)];   // points past the list repeat its last one
        const uint32_t pkg = core_list[o >> 6];
#pragma unroll 1
        for (int q0 = 0; q0 < n; q0 += kFbStep) {
            uint32_t id[kFbStep / 2];
            int cell[kFbStep / 2];
#pragma unroll
            for (int m = 0; m < kFbStep / 2; ++m) {
                const int q = q0 + 2 * m + (half >> 5);
                cell[m] = (int)((uint32_t)__shfl((int)o, q) & 63u);
                id[m] = nbr[(int64_t)(uint32_t)__shfl((int)pkg, q) * 27 + min(tap, 26)];
            }
            float v[kFbStep / 2][7];   // the tap's own value, then -x, +x, -y, +y, -z, +z
#pragma unroll
            for (int m = 0; m < kFbStep / 2; ++m) {
                // package and offset of a window point, local position + 4 per axis
                const int x = (cell[m] & 3) + tx + 4, y = ((cell[m] >> 2) & 3) + ty + 4, z = (cell[m] >> 4) + tz + 4;
                auto at = [&](int x, int y, int z) {
                    const int k = (x >> 2) + 3 * (y >> 2) + 9 * (z >> 2);
                    const int d = (x & 3) + 4 * (y & 3) + 16 * (z & 3);
                    return phi[(int64_t)(uint32_t)__shfl((int)id[m], half + k) * 64 + d];
                };
                v[m][0] = at(x, y, z);
                v[m][1] = at(x - 1, y, z);
                v[m][2] = at(x + 1, y, z);
                v[m][3] = at(x, y - 1, z);
                v[m][4] = at(x, y + 1, z);
                v[m][5] = at(x, y, z - 1);
                v[m][6] = at(x, y, z + 1);
            }
#pragma unroll
            for (int m = 0; m < kFbStep / 2; ++m)
                s_v[w][q0 + 2 * m + (half >> 5)][tap] =
                    sgrid::plane_cube_fraction(v[m][0] * inv_h, (v[m][2] - v[m][1]) * inv_2h,
                                               (v[m][4] - v[m][3]) * inv_2h, (v[m][6] - v[m][5]) * inv_2h);
        }
        __builtin_amdgcn_wave_barrier();
        if (lane < n) {
            const float *t = s_v[w][lane];
            float kw, kx, ky, kz;
            sgrid::tap_sums(
                [&](int x, int y, int z) {
                    auto far = [](int a) { return a < 0 || a > 1; };
                    const int b = far(x) ? 1 : (far(y) ? 2 : (far(z) ? 3 : 0));
                    return t[8 * b + 4 * (x > 0) + 2 * (y > 0) + (z > 0)];
                },
                0, 0, 0, kw, kx, ky, kz);
            out[o] = kw;
            out[stride + o] = kx;
            out[2 * stride + o] = ky;
            out[3 * stride + o] = kz;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Network inputs (windows of phi / h) and saturation of every core point, in
// the output order of the integrals.  unsat[o] = 1 when some tap fraction lies
// strictly between 0 and 1.
__global__ __launch_bounds__(256) void gather_windows_kernel(const float *__restrict__ phi,
                                                             const uint32_t *__restrict__ nbr,
                                                             const uint32_t *__restrict__ core_list, float inv_h,
                                                             float inv_2h, float *__restrict__ x,
                                                             uint8_t *__restrict__ unsat) {
    __shared__ float s_phi[kWinN];
    __shared__ uint32_t s_ids[27];
    __shared__ uint8_t s_sat[kVolN];
    const int64_t ci = blockIdx.x;
    stage_window(phi, nbr, core_list[ci], s_phi, s_ids);
    saturation_flags(s_phi, inv_h, inv_2h, s_sat);
    __syncthreads();
    if (x) {
        for (int e = threadIdx.x; e < 64 * kIn; e += blockDim.x) {
            const int c = e / kIn, kk = e % kIn;
            const int i = c & 3, j = (c >> 2) & 3, k = c >> 4;
            const int ox = kk % 6, oy = (kk / 6) % 6, oz = kk / 36;
            x[(ci * 64 + c) * kIn + kk] = s_phi[(i + ox) + kWin * ((j + oy) + kWin * (k + oz))] * inv_h;
        }
    }
    if (unsat && threadIdx.x < 64) {
        const int c = threadIdx.x;
        const int i = c & 3, j = (c >> 2) & 3, k = c >> 4;
        bool all = true;
        for (int oz = -1; oz <= 2; ++oz)
            for (int oy = -1; oy <= 2; ++oy)
                for (int ox = -1; ox <= 2; ++ox) {
                    const float dx = 0.5f - ox, dy = 0.5f - oy, dz = 0.5f - oz;
                    if (dx * dx + dy * dy + dz * dz >= 4.0f) continue;
                    all = all && (s_sat[(i + ox + 1) + kVol * ((j + oy + 1) + kVol * (k + oz + 1))] & 1);
                }
        unsat[ci * 64 + c] = all ? 0 : 1;
    }
}

}  // namespace

namespace sgrid {

// Gate + network over the core packages [ci0, ci_end), then the plain
// fallback over the listed points.  `fb_list` holds (ci_end - ci0) * 64
// entries; `count` is reset here.  The fallback grid is a persistent one of at
// most four workgroups per compute unit striding over the device-side count,
// so a launch costs little when few points fall back.
static sgrid_status learned_launch(const sgrid_grid *g, const float *phi, const sgrid_mlp *m, float *out,
                                   uint32_t *fb_list, uint32_t *count, int64_t ci0, int64_t ci_end, hipStream_t st) {
    hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(1), 0, st, count);
    SG_CHECK_LAUNCH("fallback counter reset");
    if (ci_end <= ci0) return SGRID_OK;
    const int64_t cells = (ci_end - ci0) * 64;
    const float inv_h = (float)(1.0 / g->h), inv_2h = (float)(0.5 / g->h);
    hipLaunchKernelGGL(learned_kernel, dim3((unsigned)((ci_end - ci0 + kLearnPkgs - 1) / kLearnPkgs)), dim3(256), 0,
                       st, m->dev(), phi, g->nbr, g->core_list, g->n_core, ci0, ci_end, inv_h, inv_2h, m->gate_tau,
                       m->kw_lo, m->kw_hi, out, fb_list, count);
    SG_CHECK_LAUNCH("learned integrals");
    const int64_t fb_blocks = std::min<int64_t>((cells + 4 * kFbPts - 1) / (4 * kFbPts), 4 * (int64_t)cu_count());
    hipLaunchKernelGGL(fallback_kernel, dim3((unsigned)fb_blocks), dim3(256), 0, st, phi, g->nbr, g->core_list,
                       g->n_core, inv_h, inv_2h, fb_list, count, out);
    SG_CHECK_LAUNCH("fallback integrals");
    return SGRID_OK;
}

sgrid_status integrals_learned(const sgrid_grid *g, const float *phi, const sgrid_mlp *model_c, float *out,
                               uint32_t *n_fallback, hipStream_t st) {
    sgrid_mlp *m = const_cast<sgrid_mlp *>(model_c);
    const int64_t cells = g->n_core * 64;
    SG_REQUIRE(g->n_core <= kMaxGrid, "too many core packages");
    sgrid_status s = mlp_ensure_fallback(m, cells);
    if (s != SGRID_OK) return s;
    s = begin_use(m, st);
    if (s != SGRID_OK) return s;
    uint32_t *count = n_fallback ? n_fallback : m->fallback + m->fallback_cap;
    s = learned_launch(g, phi, m, out, m->fallback, count, 0, g->n_core, st);
    if (s != SGRID_OK) return s;
    return end_use(m, st);
}

}  // namespace sgrid

// ---------------------------------------------------------------------------
// Learned integrals without allocation
// ---------------------------------------------------------------------------
// The fallback list lives in a fixed array in every GPU's memory (8 MiB each,
// held until the process ends): two counters padded to 256 bytes, then room
// for one chunk of kNoAllocChunk core packages' points.  Host code reaches it
// only through the address hipGetSymbolAddress returns on each device.
constexpr int64_t kNoAllocChunk = 32768;
constexpr int64_t kNoAllocWords = 64 + kNoAllocChunk * 64;
static __device__ __align__(256) uint32_t scratch[kNoAllocWords];

namespace {

constexpr int kNoAllocDevices = 64;
std::mutex g_scratch_mutex;
uint32_t *g_scratch_ptr[kNoAllocDevices] = {};

// The device address of `scratch` on the current device, looked up on the
// first call there.
sgrid_status scratch_address(int dev, uint32_t **out) {
    SG_REQUIRE(dev >= 0 && dev < kNoAllocDevices, "device %d is beyond the %d devices the library tracks", dev,
               kNoAllocDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        SG_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        SG_REQUIRE(p != nullptr, "no device address for the fallback array on device %d", dev);
        g_scratch_ptr[dev] = static_cast<uint32_t *>(p);
    }
    *out = g_scratch_ptr[dev];
    return SGRID_OK;
}

}  // namespace

extern "C" sgrid_status sgrid_compute_near_surface_integrals_noalloc(const sgrid_grid *g, const float *phi,
                                                                     const sgrid_mlp *model, float *out,
                                                                     uint32_t *n_fallback, void *stream) {
    sgrid::clear_error();
    SG_REQUIRE(g != nullptr, "grid is NULL");
    SG_REQUIRE(model != nullptr, "model is NULL (the plain integrals allocate nothing: use "
                                 "sgrid_compute_near_surface_integrals)");
    SG_REQUIRE(phi != nullptr, "phi is NULL");
    SG_REQUIRE(out != nullptr || g->n_core == 0, "out is NULL");
    SG_REQUIRE(sg_aligned(phi, 16) && sg_aligned(out, 16), "phi / out must be 16-byte aligned");
    SG_REQUIRE(g->n_core * 64 <= (int64_t)UINT32_MAX, "%lld core packages: point indices exceed 32 bits",
               (long long)g->n_core);
    int dev = 0;
    SG_CHECK_HIP(hipGetDevice(&dev));
    SG_REQUIRE(g->device == dev && model->device == dev,
               "grid (device %d) and model (device %d) must live on the current device %d", g->device,
               model->device, dev);
    uint32_t *sc = nullptr;
    sgrid_status s = scratch_address(dev, &sc);
    if (s != SGRID_OK) return s;
    hipStream_t st = sg_stream(stream);
    s = sgrid::begin_use(model, st);
    if (s != SGRID_OK) return s;
    uint32_t *chunk_count = sc, *total = n_fallback ? n_fallback : sc + 1, *list = sc + 64;
    hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(1), 0, st, total);
    SG_CHECK_LAUNCH("fallback total reset");
    for (int64_t ci0 = 0; ci0 < g->n_core; ci0 += kNoAllocChunk) {
        const int64_t ci_end = std::min<int64_t>(ci0 + kNoAllocChunk, g->n_core);
        s = sgrid::learned_launch(g, phi, model, out, list, chunk_count, ci0, ci_end, st);
        if (s != SGRID_OK) return s;
        hipLaunchKernelGGL(add_u32_kernel, dim3(1), dim3(1), 0, st, total, (const uint32_t *)chunk_count);
        SG_CHECK_LAUNCH("fallback total");
    }
    return sgrid::end_use(model, st);
}

sgrid_status sgrid::launch_zero_u32(uint32_t *p, hipStream_t st) {
    hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(1), 0, st, p);
    SG_CHECK_LAUNCH("counter reset");
    return SGRID_OK;
}

extern "C" sgrid_status sgrid_gather_windows(const sgrid_grid *g, const float *phi, float *x_dev, uint8_t *unsat_dev,
                                             void *stream) {
    sgrid::clear_error();
    SG_REQUIRE(g != nullptr && phi != nullptr, "grid or phi is NULL");
    SG_REQUIRE(sg_aligned(phi, 16) && sg_aligned(x_dev, 4), "phi / x misaligned");
    if (g->n_core == 0) return SGRID_OK;
    SG_REQUIRE(g->n_core <= kMaxGrid, "too many core packages");
    hipLaunchKernelGGL(gather_windows_kernel, dim3((unsigned)g->n_core), dim3(256), 0, sg_stream(stream), phi, g->nbr,
                       g->core_list, (float)(1.0 / g->h), (float)(0.5 / g->h), x_dev, unsat_dev);
    SG_CHECK_LAUNCH("gather windows");
    return SGRID_OK;
}
