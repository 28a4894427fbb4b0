// Steps of the tiled form on the matrix cores: C(m, n) = sum_k A[k][m] B[k][n]
// with both operands in memory as the layout pass leaves them ([K][M] and
// [K][N]), C written through offset tables into its consumer's layout.
// Shared by the per-step launch (tile.hip) and the batch's item kernels
// (queue.hip), so that a step gives the same result bit for bit in all.
//
// With FP64 results of FP32 or BF16 operands the elements are widened as they
// are read, and products and sums are FP64.
//
// A wave computes four 16 x 16 blocks (1024 results) by itself: 32 x 32, or
// 64 x 16 or 16 x 64 where M or N is small.  A lane's
// operand for a matrix instruction is one element: sixteen lanes read
// sixteen neighbours of a row of A (or B), so the fragments come straight
// from global memory in whole segments, with no LDS (which leaves the CU to
// a fused-kernel workgroup that holds most of it) and no barrier; the
// fragments of the next K chunk are read while the current one is
// multiplied.  The table-driven step this replaces reads both operands and
// two table entries for every single product: a 576 x 36 x 3456 step in FP32
// took 65 us alone on the chip, the levels that hold the products of 25 random
// networks (1.2 G products in FP32) 775 us in all, now 271 us; the queue of a
// BF16 batch of 60-vertex rings went from 721 to 382 us.
#pragma once

#include "kern_common.hpp"
#include "mfma_dev.hpp"

namespace htn {
namespace kern {

// One K chunk of 4 KU values: fragments of WM row and WN column blocks.
template <typename T, int KU, int WM, int WN>
struct TileFrag {
    T a[KU][WM], b[KU][WN];
    template <bool TAIL, typename TA, typename TB>
    __device__ __forceinline__ void load(const TA *__restrict__ A, const TB *__restrict__ B, const int (&om)[WM],
                                         const int (&on)[WN], int M, int N, int k0, int kend, int lk) {
        const TA *pa = A + (int64_t)k0 * M;
        const TB *pb = B + (int64_t)k0 * N;
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int k = 4 * u + lk;
            // past the range: the products are zero (both factors, so that
            // no infinity meets a zero), read from the range's first row
            const bool ok = !TAIL || k0 + k < kend;
            const int ra = ok ? k * M : 0, rb = ok ? k * N : 0;
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                a[u][i] = to_compute<T>(pa[ra + om[i]]);
                if (TAIL && !ok) a[u][i] = 0;
            }
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                b[u][j] = to_compute<T>(pb[rb + on[j]]);
                if (TAIL && !ok) b[u][j] = 0;
            }
        }
    }
};

template <typename T, typename TA, typename TB, int WM, int WN>
__device__ __forceinline__ void tile_unit(const TA *__restrict__ A, const TB *__restrict__ B, void *C, int tc,
                                          const int2 *__restrict__ tab, const TileArgs &t, int w) {
    typedef MfmaOp<T> Op;
    constexpr int KU = sizeof(T) == 4 ? 8 : 4, KC = 4 * KU;
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const int tiles = t.tiles_m * t.tiles_n;
    const int kz = w / tiles, r = w - kz * tiles;
    const int tm = r / t.tiles_n, tn = r - tm * t.tiles_n;
    const int m0 = tm * 16 * WM, n0 = tn * 16 * WN;
    const int kend = min(t.K, (kz + 1) * t.kper);
    int k0 = kz * t.kper;
    int om[WM], on[WN];
    // (rows and columns past the matrix repeat the last one; not stored)
#pragma unroll
    for (int i = 0; i < WM; ++i) om[i] = min(m0 + 16 * i + lr, t.M - 1);
#pragma unroll
    for (int j = 0; j < WN; ++j) on[j] = min(n0 + 16 * j + lr, t.N - 1);
    typename Op::acc tot[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) tot[i][j] = typename Op::acc{0, 0, 0, 0};
    // Sixteen terms are accumulated by the matrix core before they join the
    // result's running sum: a chain of FP32 additions K long would lose more
    // than the lanes' partial sums of a table-driven step.
    auto mult = [&](const TileFrag<T, KU, WM, WN> &f) {
#pragma unroll
        for (int q = 0; q < KU; q += 4) {
            typename Op::acc acc[WM][WN];
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j) acc[i][j] = typename Op::acc{0, 0, 0, 0};
#pragma unroll
            for (int u = q; u < q + 4; ++u)
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) acc[i][j] = Op::mma(f.a[u][i], f.b[u][j], acc[i][j]);
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) tot[i][j][e] += acc[i][j][e];
        }
    };
    TileFrag<T, KU, WM, WN> f, g;
    if (k0 + KC <= kend) {
        f.template load<false>(A, B, om, on, t.M, t.N, k0, kend, lk);
        for (; k0 + 2 * KC <= kend; k0 += KC) {
            g.template load<false>(A, B, om, on, t.M, t.N, k0 + KC, kend, lk);
            mult(f);
            f = g;
        }
        if (k0 + KC < kend) {
            g.template load<true>(A, B, om, on, t.M, t.N, k0 + KC, kend, lk);
            mult(f);
            mult(g);
        } else {
            mult(f);
        }
    } else if (k0 < kend) {
        f.template load<true>(A, B, om, on, t.M, t.N, k0, kend, lk);
        mult(f);
    }
    int cn[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j) cn[j] = tab[t.t_cn + on[j]].x;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = m0 + 16 * i + Op::row(lane, e);
            if (m >= t.M) continue;
            const int cm = tab[t.t_cm + m].x;
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                if (n0 + 16 * j + lr >= t.N) continue;
                const int64_t o = (int64_t)kz * t.total + cm + cn[j];
                if constexpr (sizeof(T) == 8) {  // FP64 results
                    ((double *)C)[o] = tot[i][j][e];
                } else {
                    if (tc == 2)
                        ((bf16_t *)C)[o] = f2bf(tot[i][j][e]);
                    else
                        ((float *)C)[o] = tot[i][j][e];
                }
            }
        }
}

// Wave tile w of the step: ((kz * tiles_m + tm) * tiles_n + tn).
template <typename T, typename TA, typename TB>
__device__ __forceinline__ void tile_wave(const void *A, const void *B, void *C, int tc, const int2 *__restrict__ tab,
                                          const TileArgs &t, int w) {
    if (w >= t.tiles_m * t.tiles_n * t.ksplit) return;
    if (t.shape == 0)
        tile_unit<T, TA, TB, 2, 2>((const TA *)A, (const TB *)B, C, tc, tab, t, w);
    else if (t.shape == 1)
        tile_unit<T, TA, TB, 4, 1>((const TA *)A, (const TB *)B, C, tc, tab, t, w);
    else
        tile_unit<T, TA, TB, 1, 4>((const TA *)A, (const TB *)B, C, tc, tab, t, w);
}

__device__ __forceinline__ void tile_wave_any(const void *A, int ta, const void *B, int tb, void *C, int tc,
                                              const int2 *__restrict__ tab, const TileArgs &t, int w) {
    if (ta == 0)
        tile_wave<double, double, double>(A, B, C, tc, tab, t, w);
    else if (tc == 0 && ta == 1 && tb == 1)
        tile_wave<double, float, float>(A, B, C, tc, tab, t, w);
    else if (tc == 0 && ta == 2 && tb == 2)
        tile_wave<double, bf16_t, bf16_t>(A, B, C, tc, tab, t, w);
    else if (tc == 0 && ta == 2)
        tile_wave<double, bf16_t, float>(A, B, C, tc, tab, t, w);
    else if (tc == 0)
        tile_wave<double, float, bf16_t>(A, B, C, tc, tab, t, w);
    else if (ta == 1 && tb == 1)
        tile_wave<float, float, float>(A, B, C, tc, tab, t, w);
    else if (ta == 2 && tb == 2)
        tile_wave<float, bf16_t, bf16_t>(A, B, C, tc, tab, t, w);
    else if (ta == 2)
        tile_wave<float, bf16_t, float>(A, B, C, tc, tab, t, w);
    else
        tile_wave<float, float, bf16_t>(A, B, C, tc, tab, t, w);
}

}  // namespace kern
}  // namespace htn
