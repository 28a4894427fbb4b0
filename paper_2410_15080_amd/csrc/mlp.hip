// Cost-model MLP kernels: forward, gradients, Adam.
//
// The model maps the feature vector of one kernel step to the natural log
// of its duration:  h1 = relu(W1 x + b1), h2 = relu(W2 h1 + b2),
// y = w3 . h2 + b3, with F inputs, H = 64 hidden units per layer, FP32
// throughout.  Flat parameter layout: W1 [H][F], b1 [H], W2 [H][H], b2 [H],
// w3 [H], b3 [1].  Training loss: mean squared error over the batch.
//
// Every product is a small matrix product over a tile of 64 samples (16 per
// wave) on the FP32 matrix cores (16x16x4).  Lane l = 16 g + i of a wave
// holds sample i of the wave's 16 and, of a 16-row block b, rows
// 16 b + 4 g + r (r = 0..3): the layout in which the instruction returns
// its result.  The summed index of the next product is taken in the same
// order (step (b, r) sums rows 16 b + 4 g + r over g), so a layer's result
// is the next layer's operand without a shuffle.
//
// What bounds them: 14 227 samples are 0.2 GFLOP forward and 0.4 more for
// the gradients (5 us at the FP32 matrix rate); the rest is one pass of
// latencies (weights into LDS, a tile's chain of layers).  One thread per
// sample forward (56 workgroups) and one thread per parameter summing all
// samples (23 workgroups, a serial chain of 14 227 loads) took 38 us and
// 3 900 us; figures of the present kernels stand at each of them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "htn.h"
#include "kernels.hpp"

namespace htn {
namespace kern {

namespace {
constexpr int MF = HTN_MODEL_FEATURES, MH = HTN_MODEL_HIDDEN;
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + MH * MF;
constexpr int OFF_W2 = OFF_B1 + MH;
constexpr int OFF_B2 = OFF_W2 + MH * MH;
constexpr int OFF_W3 = OFF_B2 + MH;
constexpr int OFF_B3 = OFF_W3 + MH;
constexpr int NPARAM = OFF_B3 + 1;
constexpr int TPB = 256;
constexpr int kTile = 64;       // samples per workgroup pass
constexpr int kFwdBlocks = 1024;
constexpr int LDX = 36;         // padded row of W1 in LDS (features 0..31, zero beyond MF)
constexpr int LDT = 68;         // padded row of a 64-wide array in LDS: 16-byte
                                // aligned, and rows four apart fall on other banks
static_assert(MH == 64 && MF <= 32, "the tiles below");

typedef float f4 __attribute__((ext_vector_type(4)));

struct Weights {
    float w1[MH * LDX];
    float w2[MH * LDT];
    float b1[MH], b2[MH], w3[MH];
    float b3, pad[3];
};

__device__ __forceinline__ void load_weights(Weights &w, const float *__restrict__ prm) {
    for (int e = threadIdx.x; e < MH * 32; e += TPB) {
        const int j = e >> 5, f = e & 31;
        w.w1[j * LDX + f] = f < MF ? prm[OFF_W1 + j * MF + f] : 0.0f;
    }
    for (int e = threadIdx.x; e < MH * MH; e += TPB) w.w2[(e >> 6) * LDT + (e & 63)] = prm[OFF_W2 + e];
    if (threadIdx.x < MH) {
        w.b1[threadIdx.x] = prm[OFF_B1 + threadIdx.x];
        w.b2[threadIdx.x] = prm[OFF_B2 + threadIdx.x];
        w.w3[threadIdx.x] = prm[OFF_W3 + threadIdx.x];
    }
    if (threadIdx.x == 0) w.b3 = prm[OFF_B3];
}

__device__ __forceinline__ f4 mma(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Features 16 b + 4 g + r of the lane's sample (0 beyond MF and for ok = false).
__device__ __forceinline__ void load_x(const float *__restrict__ x, int64_t row, bool ok, int g, float xv[2][4]) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int f = 16 * b + 4 * g + r;
            xv[b][r] = ok && f < MF ? x[row * MF + f] : 0.0f;
        }
}

// z1, z2 (pre-activations) and y of the lane's sample; the terms of a
// unit's sum start from its bias.
__device__ __forceinline__ float forward(const Weights &w, const float xv[2][4], int li, int g, f4 z1[4], f4 z2[4]) {
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        z1[o] = *(const f4 *)(w.b1 + 16 * o + 4 * g);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const f4 a = *(const f4 *)(w.w1 + (16 * o + li) * LDX + 16 * b + 4 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) z1[o] = mma(a[r], xv[b][r], z1[o]);
        }
    }
    float y = 0.0f;
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        z2[o] = *(const f4 *)(w.b2 + 16 * o + 4 * g);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const f4 a = *(const f4 *)(w.w2 + (16 * o + li) * LDT + 16 * b + 4 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) z2[o] = mma(a[r], fmaxf(z1[b][r], 0.0f), z2[o]);
        }
        const f4 w3 = *(const f4 *)(w.w3 + 16 * o + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) y = fmaf(w3[r], fmaxf(z2[o][r], 0.0f), y);
    }
    y += __shfl_xor(y, 16);
    y += __shfl_xor(y, 32);
    return y + w.b3;
}
}  // namespace

int64_t model_param_count() { return NPARAM; }

// Predictions of n samples (sample s reads row idx[s] of x when idx is given).
// 14 227 samples: 38.3 -> 7.8 us (223 workgroups of 64 samples instead of 56
// of 256; a wave waits mostly for the weights on their way into LDS).
__global__ __launch_bounds__(TPB) void k_mlp_fwd(const float *__restrict__ prm, const float *__restrict__ x,
                                                const int32_t *__restrict__ idx, int n, float *__restrict__ y) {
    __shared__ __align__(16) Weights w;
    load_weights(w, prm);
    __syncthreads();
    const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
    for (int64_t s = (int64_t)blockIdx.x * kTile + 16 * (threadIdx.x >> 6) + li; s - li < n;
         s += (int64_t)gridDim.x * kTile) {
        const bool ok = s < n;
        const int64_t row = ok ? (idx ? idx[s] : s) : 0;
        float xv[2][4];
        f4 z1[4], z2[4];
        load_x(x, row, ok, g, xv);
        const float v = forward(w, xv, li, g, z1, z2);
        if (ok && g == 0) y[s] = v;
    }
}

// One workgroup's share of the gradient: part[block][NPARAM] and, in the
// slot after the parameters, its sum of squared errors.  Per tile of 64
// samples: forward, then
//   dy_s = 2 (y_s - t_s) / n,  dz2 = dy_s w3 * [z2 > 0],  dz1 = W2^T dz2 * [z1 > 0],
// each wave its 16 samples; the tile's h1, dz2, dz1 and x go through LDS
// as [unit][sample] so that the weight gradients are products summed over
// the 64 samples, wave w taking rows 16 w .. 16 w + 15 of both.  The sums
// run in a fixed order (the gradients are bit-reproducible).  14 227
// samples: 17.1 us and 3.9 us for the reduction, against 3 960 us for the
// five launches with one thread per parameter; the whole gradient call and a
// forward 3 985 -> 28.4 us, its error against 64 bits 1.8e-6 -> 2.7e-7.
struct GradTile {
    Weights w;
    float h1[MH * LDT], d2[MH * LDT], d1[MH * LDT], x[32 * LDT];
    float bias[4][3 * MH + 2];  // per wave: b1, b2, w3, then b3 and the loss
};

__global__ __launch_bounds__(TPB) void k_mlp_grad(const float *__restrict__ prm, const float *__restrict__ x,
                                                 const float *__restrict__ t, const int32_t *__restrict__ idx, int n,
                                                 float scale, float *__restrict__ part) {
    extern __shared__ __align__(16) unsigned char mlp_lds[];
    GradTile &L = *reinterpret_cast<GradTile *>(mlp_lds);
    load_weights(L.w, prm);
    const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
    f4 gw2[4], gw1[2], gb1[4], gb2[4], gw3[4];
#pragma unroll
    for (int o = 0; o < 4; ++o) gw2[o] = gb1[o] = gb2[o] = gw3[o] = f4{0, 0, 0, 0};
    gw1[0] = gw1[1] = f4{0, 0, 0, 0};
    float gb3 = 0.0f, loss = 0.0f;
    const int st = 16 * wave + li;  // the lane's sample in the tile
    for (int64_t s0 = (int64_t)blockIdx.x * kTile; s0 < n; s0 += (int64_t)gridDim.x * kTile) {
        __syncthreads();  // weights loaded; the last tile's arrays read
        const int64_t s = s0 + st;
        const bool ok = s < n;
        const int64_t row = ok ? (idx ? idx[s] : s) : 0;
        float xv[2][4];
        f4 z1[4], z2[4], d1[4];
        load_x(x, row, ok, g, xv);
        const float y = forward(L.w, xv, li, g, z1, z2);
        const float e = ok ? y - t[row] : 0.0f;
        const float dy = scale * e;
        if (g == 0) {
            gb3 += dy;
            loss = fmaf(e, e, loss);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) L.x[(16 * b + 4 * g + r) * LDT + st] = xv[b][r];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const f4 w3 = *(const f4 *)(L.w.w3 + 16 * o + 4 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gw3[o][r] = fmaf(dy, fmaxf(z2[o][r], 0.0f), gw3[o][r]);
                const float d = ok && z2[o][r] > 0.0f ? dy * w3[r] : 0.0f;
                z2[o][r] = d;  // dz2 from here on
                gb2[o][r] += d;
                L.d2[(16 * o + 4 * g + r) * LDT + st] = d;
                L.h1[(16 * o + 4 * g + r) * LDT + st] = ok ? fmaxf(z1[o][r], 0.0f) : 0.0f;
            }
        }
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            d1[o] = f4{0, 0, 0, 0};
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    d1[o] = mma(L.w.w2[(16 * b + 4 * g + r) * LDT + 16 * o + li], z2[b][r], d1[o]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float d = z1[o][r] > 0.0f ? d1[o][r] : 0.0f;
                gb1[o][r] += d;
                L.d1[(16 * o + 4 * g + r) * LDT + st] = d;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f4 a2 = *(const f4 *)(L.d2 + (16 * wave + li) * LDT + 16 * q + 4 * g);
            const f4 a1 = *(const f4 *)(L.d1 + (16 * wave + li) * LDT + 16 * q + 4 * g);
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const f4 h = *(const f4 *)(L.h1 + (16 * o + li) * LDT + 16 * q + 4 * g);
#pragma unroll
                for (int r = 0; r < 4; ++r) gw2[o] = mma(a2[r], h[r], gw2[o]);
            }
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const f4 xt = *(const f4 *)(L.x + (16 * o + li) * LDT + 16 * q + 4 * g);
#pragma unroll
                for (int r = 0; r < 4; ++r) gw1[o] = mma(a1[r], xt[r], gw1[o]);
            }
        }
    }
    float *out = part + (int64_t)blockIdx.x * (NPARAM + 1);
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[OFF_W2 + (16 * wave + 4 * g + r) * MH + 16 * o + li] = gw2[o][r];
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (16 * o + li < MF) out[OFF_W1 + (16 * wave + 4 * g + r) * MF + 16 * o + li] = gw1[o][r];
    // biases and w3: over a wave's 16 samples, then over the waves in order
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) {
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gb1[o][r] += __shfl_xor(gb1[o][r], m);
                gb2[o][r] += __shfl_xor(gb2[o][r], m);
                gw3[o][r] += __shfl_xor(gw3[o][r], m);
            }
        gb3 += __shfl_xor(gb3, m);
        loss += __shfl_xor(loss, m);
    }
    if (li == 0) {
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = 16 * o + 4 * g + r;
                L.bias[wave][j] = gb1[o][r];
                L.bias[wave][MH + j] = gb2[o][r];
                L.bias[wave][2 * MH + j] = gw3[o][r];
            }
        if (g == 0) {
            L.bias[wave][3 * MH] = gb3;
            L.bias[wave][3 * MH + 1] = loss;
        }
    }
    __syncthreads();
    if (threadIdx.x < 3 * MH + 2) {
        const int q = threadIdx.x;
        const float v = (L.bias[0][q] + L.bias[1][q]) + (L.bias[2][q] + L.bias[3][q]);
        const int p = q < MH          ? OFF_B1 + q
                      : q < 2 * MH    ? OFF_B2 + q - MH
                      : q < 3 * MH    ? OFF_W3 + q - 2 * MH
                      : q == 3 * MH   ? OFF_B3
                                      : NPARAM;
        out[p] = v;
    }
}

// Adam (Kingma & Ba): m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// p -= lr * (m / (1-b1^t)) / (sqrt(v / (1-b2^t)) + eps).
struct AdamArgs {
    float *p, *m, *v;
    float lr, b1, b2, c1, c2, eps;
};

__device__ __forceinline__ void adam_one(const AdamArgs &a, int i, float gi) {
    const float mi = a.b1 * a.m[i] + (1.0f - a.b1) * gi;
    const float vi = a.b2 * a.v[i] + (1.0f - a.b2) * gi * gi;
    a.m[i] = mi;
    a.v[i] = vi;
    a.p[i] -= a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
}

// Sums the workgroups' shares: 64 parameters per workgroup, 16 waves each
// taking every 16th share, then the waves in order.  With a.p set the Adam
// step follows at once (a training step is two launches).
constexpr int kRedWaves = 16;
__global__ __launch_bounds__(64 * kRedWaves) void k_mlp_reduce(const float *__restrict__ part, int n_part, int n,
                                                               float *__restrict__ grad, float *__restrict__ loss,
                                                               const AdamArgs a) {
    __shared__ float red[kRedWaves][64];
    const int q = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + q;
    float acc = 0.0f;
    if (p <= NPARAM) {
#pragma unroll 4
        for (int b = wave; b < n_part; b += kRedWaves) acc += part[(int64_t)b * (NPARAM + 1) + p];
    }
    red[wave][q] = acc;
    __syncthreads();
    if (wave != 0 || p > NPARAM) return;
    float v = red[0][q];
#pragma unroll
    for (int w = 1; w < kRedWaves; ++w) v += red[w][q];
    if (p == NPARAM) {
        if (loss) *loss = v / (float)n;
        return;
    }
    grad[p] = v;
    if (a.p) adam_one(a, p, v);
}

__global__ __launch_bounds__(TPB) void k_adam(const float *__restrict__ g, const AdamArgs a) {
    const int i = blockIdx.x * TPB + threadIdx.x;
    if (i < NPARAM) adam_one(a, i, g[i]);
}

hipError_t launch_mlp_forward(const float *prm, const float *x, const int32_t *idx, int n, float *y, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>(((int64_t)n + kTile - 1) / kTile, kFwdBlocks);
    hipLaunchKernelGGL(k_mlp_fwd, dim3(blocks), dim3(TPB), 0, st, prm, x, idx, n, y);
    return hipGetLastError();
}

// One workgroup per CU (its tile arrays take 90 KB of LDS).
static constexpr int kGradBlocks = 256;
static int grad_blocks(int64_t n) { return (int)std::min<int64_t>((n + kTile - 1) / kTile, kGradBlocks); }

int64_t mlp_part_floats(int64_t n) { return (int64_t)grad_blocks(n) * (NPARAM + 1); }

static AdamArgs adam_args(const MlpAdam *a) {
    AdamArgs r{};
    if (!a) return r;
    r.p = a->p;
    r.m = a->m;
    r.v = a->v;
    r.lr = a->lr;
    r.b1 = 0.9f;
    r.b2 = 0.999f;
    r.eps = 1e-8f;
    r.c1 = (float)(1.0 / (1.0 - std::pow(0.9, (double)a->step)));
    r.c2 = (float)(1.0 / (1.0 - std::pow(0.999, (double)a->step)));
    return r;
}

hipError_t launch_mlp_gradients(const float *prm, const float *x, const float *t, const int32_t *idx, int n,
                                float *part, float *grad, float *loss, const MlpAdam *adam, hipStream_t st) {
    if (n <= 0) return hipErrorInvalidValue;
    const hipError_t e = hipFuncSetAttribute((const void *)k_mlp_grad, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)sizeof(GradTile));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e;
    }
    const int blocks = grad_blocks(n);
    hipLaunchKernelGGL(k_mlp_grad, dim3(blocks), dim3(TPB), sizeof(GradTile), st, prm, x, t, idx, n, 2.0f / (float)n,
                       part);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NPARAM + 1 + 63) / 64), dim3(64 * kRedWaves), 0, st, part, blocks, n, grad,
                       loss, adam_args(adam));
    return hipGetLastError();
}

hipError_t launch_adam(const MlpAdam &a, const float *g, hipStream_t st) {
    hipLaunchKernelGGL(k_adam, dim3((NPARAM + TPB - 1) / TPB), dim3(TPB), 0, st, g, adam_args(&a));
    return hipGetLastError();
}

}  // namespace kern
}  // namespace htn
