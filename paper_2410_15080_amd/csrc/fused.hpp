// The fused whole-network kernel (k_fused) and its step routines.  One
// workgroup contracts an entire network: a program image (built by the
// planner) is copied into LDS and interpreted; operands and intermediates
// stay in LDS where they fit (else in the network's workspace); each
// pairwise step is a register-tiled product or a table-driven reduction;
// the last step writes the result.  One launch serves a batch of networks
// (one workgroup each).  Each workgroup size is instantiated in its own
// translation unit (fused_b*.hip).
//
// What bounds it: latency.  A network is 6-10 dependent phases of a few
// hundred multiplications per thread, so what a phase costs besides its
// arithmetic decides: finding and decoding the wave's step, the copies for
// the next phase, the offsets of the results, the barrier.
#pragma once

#include <type_traits>

#include "kern_common.hpp"

namespace htn {
namespace kern {

// ----------------------------------------------------------------- k_fused

// Program words of a step, word i in lane i (words 64.. in a second
// register): one LDS read brings them all, and a wave-uniform read is then
// one lane read.  Reading each word where it lies in LDS instead made
// every field a round trip of 130 cycles, and the fields' use a chain of
// them: 900-3200 cycles to find a wave's step, 4000-6000 for the offsets of
// a 24 x 16 result.
struct StepWords {
    int32_t r, d;  // the step's fields; the digit descriptors of a tiled step
    __device__ __forceinline__ StepWords(const int32_t *img, int n_words, int off, int lane) {
        r = off + lane < n_words ? img[off + lane] : 0;
        d = off + 15 + lane < n_words ? img[off + 15 + lane] : 0;
    }
    __device__ __forceinline__ int32_t operator()(int i) const { return __builtin_amdgcn_readlane(r, i); }
    __device__ __forceinline__ int32_t digit(int i) const { return __builtin_amdgcn_readlane(d, i); }
};

// Pointers of known address spaces, so that operands and results in LDS are
// read and written by LDS instructions (a pointer that may be either is
// accessed through the slower flat path).
template <typename T>
using LdsPtr = __attribute__((address_space(3))) T *;
template <typename T>
using GlobalPtr = __attribute__((address_space(1))) T *;

// Where a step's results go.
template <typename T>
struct Dest {
    bool in_lds;
    LdsPtr<T> l;
    GlobalPtr<T> g;
    __device__ __forceinline__ void put(int o, T v) const {
        if (in_lds)  // wave-uniform
            l[o] = v;
        else
            g[o] = v;
    }
};

// The next NB terms of one output's sum from (sh, sl) on, products in pv[]
// (0 past the end); (sh, sl) advances by NB strides.
template <int NB, typename ACC, bool UNARY, typename P>
__device__ __forceinline__ void next_terms(P a0, P b0, const int2 *tsh, const int2 *tsl, int &sh, int &sl, int dq,
                                           int dr, int n_shi, int n_slo, ACC (&pv)[NB]) {
    int hv[NB], lv[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        hv[u] = sh;
        lv[u] = sl;
        sh += dq;
        sl += dr;
        if (sl >= n_slo) {
            sl -= n_slo;
            ++sh;
        }
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const bool ok = hv[u] < n_shi;
        const int2 h = tsh[ok ? hv[u] : 0], l = tsl[lv[u]];
        ACC q = (ACC)a0[h.x + l.x];
        if constexpr (!UNARY) q *= (ACC)b0[h.y + l.y];
        pv[u] = ok ? q : ACC(0);
    }
}

// Sum over the summed index space (n_shi x n_slo, two-level tables) of one
// output, visiting s = start, start + stride, ... in (sh, sl) form with
// stride = dq * n_slo + dr (dr < n_slo), `terms` of them at most per lane.
// Long sums read 16 terms ahead of their additions (operands outside LDS
// take 1000 cycles and more: a sum of 3456 terms by 16 lanes took 164 000
// cycles with 4 in flight).  Plain sums keep four independent partial sums
// (term t in t mod 4) whatever the number in flight; compensated ones are
// added in order.
template <typename ACC, bool COMP, bool UNARY, typename P>
__device__ __forceinline__ void strided_sum(P a0, P b0, const int2 *tsh, const int2 *tsl, int sh, int sl, int dq,
                                            int dr, int n_shi, int n_slo, int terms, ACC &s, ACC &c) {
    if constexpr (!COMP) {
        ACC s1 = 0, s2 = 0, s3 = 0;
        for (; terms > 8; terms -= 16) {  // terms: the same for every lane
            ACC pv[16];
            next_terms<16, ACC, UNARY>(a0, b0, tsh, tsl, sh, sl, dq, dr, n_shi, n_slo, pv);
#pragma unroll
            for (int u = 0; u < 16; u += 4) {
                s += pv[u];
                s1 += pv[u + 1];
                s2 += pv[u + 2];
                s3 += pv[u + 3];
            }
        }
        for (; terms > 0; terms -= 4) {
            ACC pv[4];
            next_terms<4, ACC, UNARY>(a0, b0, tsh, tsl, sh, sl, dq, dr, n_shi, n_slo, pv);
            s += pv[0];
            s1 += pv[1];
            s2 += pv[2];
            s3 += pv[3];
        }
        s += (s1 + s2) + s3;
    } else {
        while (sh < n_shi) {
            ACC pv[8];
            const int h0 = sh, l0 = sl;
            next_terms<8, ACC, UNARY>(a0, b0, tsh, tsl, sh, sl, dq, dr, n_shi, n_slo, pv);
            int h = h0, l = l0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (h < n_shi) accum<COMP>(s, c, pv[u]);
                h += dq;
                l += dr;
                if (l >= n_slo) {
                    l -= n_slo;
                    ++h;
                }
            }
        }
    }
}

// Table-driven step.  Threads tid = 0..nthr-1 of the step's waves run it; R ==
// nthr (the whole workgroup per output) is planned only when the step owns the
// workgroup (nthr == BLK), since it synchronises every wave.
template <int BLK, typename ACC, bool COMP, bool UNARY, typename TOUT, typename P>
__device__ __forceinline__ void fstep(P A, P B, const Dest<TOUT> &C, const int2 *__restrict__ tab,
                                      const StepWords &p, ACC *scratch, const int tid, const int nthr) {
    const int n_ohi = p(4), n_olo = p(5), n_shi = p(6), n_slo = p(7);
    const int2 *toh = tab + p(8);
    const int2 *tol = tab + p(9);
    const int2 *tsh = tab + p(10);
    const int2 *tsl = tab + p(11);
    const int R = p(12);
    const int n_out = n_ohi * n_olo;
    int log2R = 0;
    while ((1 << log2R) < R) ++log2R;
    const int terms = (n_shi * n_slo + R - 1) >> log2R;  // of one lane, at most
    if (R == BLK && nthr == BLK) {
        // whole workgroup per output (tiny outputs, long sums)
        const int dq = BLK / n_slo, dr = BLK - dq * n_slo;
        const int sh0 = tid / n_slo, sl0 = tid - sh0 * n_slo;
        for (int o = 0; o < n_out; ++o) {
            const int oh = o / n_olo, ol = o - oh * n_olo;  // wave-uniform
            const int2 x = toh[oh], y = tol[ol];
            const P a0 = A + (x.x + y.x);
            P b0 = B;
            if constexpr (!UNARY) b0 = B + (x.y + y.y);
            ACC s = 0, c = 0;
            strided_sum<ACC, COMP, UNARY>(a0, b0, tsh, tsl, sh0, sl0, dq, dr, n_shi, n_slo, terms, s, c);
            lane_reduce<COMP>(s, c, 64);
            if ((tid & 63) == 0) {
                scratch[2 * (tid >> 6)] = s;
                scratch[2 * (tid >> 6) + 1] = c;
            }
            __syncthreads();
            if (tid == 0) {
                ACC ts = scratch[0], tc = scratch[1];
                for (int w = 1; w < BLK / 64; ++w) combine<COMP>(ts, tc, scratch[2 * w], scratch[2 * w + 1]);
                C.put(o, st_cvt<TOUT>(COMP ? ts + tc : ts));
            }
            __syncthreads();
        }
        return;
    }
    const int groups = nthr >> log2R;
    const int gi = tid >> log2R, sub = tid & (R - 1);
    const int dq = R / n_slo, dr = R - dq * n_slo;
    // output o = oh * n_olo + ol, advanced by `groups` per pass without a
    // division (one per thread up front)
    const int oq = groups / n_olo, orr = groups - oq * n_olo;
    int oh = gi / n_olo, ol = gi - oh * n_olo;
    const int sh0 = sub / n_slo, sl0 = sub - sh0 * n_slo;
    for (int o0 = 0; o0 < n_out; o0 += groups) {
        const int o = o0 + gi;
        const bool active = o < n_out;
        ACC s = 0, c = 0;
        if (active) {
            const int2 x = toh[oh], y = tol[ol];
            const P a0 = A + (x.x + y.x);
            P b0 = B;
            if constexpr (!UNARY) b0 = B + (x.y + y.y);
            if (R == 1) {
                ACC s1 = 0, s2 = 0, s3 = 0;
                for (int sh = 0; sh < n_shi; ++sh) {
                    const int2 h = tsh[sh];
                    const P a1 = a0 + h.x;
                    P b1 = b0;
                    if constexpr (!UNARY) b1 = b0 + h.y;
                    int sl = 0;
                    if constexpr (!COMP) {
                        // four independent partial sums (ILP), up to 16
                        // terms in flight
                        for (; sl + 16 <= n_slo; sl += 16) {
                            ACC q[16];
#pragma unroll
                            for (int u = 0; u < 16; ++u) {
                                const int2 l = tsl[sl + u];
                                q[u] = (ACC)a1[l.x];
                                if constexpr (!UNARY) q[u] *= (ACC)b1[l.y];
                            }
#pragma unroll
                            for (int u = 0; u < 16; u += 4) {
                                s += q[u];
                                s1 += q[u + 1];
                                s2 += q[u + 2];
                                s3 += q[u + 3];
                            }
                        }
                        for (; sl + 4 <= n_slo; sl += 4) {
                            ACC q[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const int2 l = tsl[sl + u];
                                q[u] = (ACC)a1[l.x];
                                if constexpr (!UNARY) q[u] *= (ACC)b1[l.y];
                            }
                            s += q[0];
                            s1 += q[1];
                            s2 += q[2];
                            s3 += q[3];
                        }
                    }
                    for (; sl < n_slo; ++sl) {
                        const int2 l = tsl[sl];
                        ACC p = (ACC)a1[l.x];
                        if constexpr (!UNARY) p *= (ACC)b1[l.y];
                        accum<COMP>(s, c, p);
                    }
                }
                s += (s1 + s2) + s3;
            } else {
                strided_sum<ACC, COMP, UNARY>(a0, b0, tsh, tsl, sh0, sl0, dq, dr, n_shi, n_slo, terms, s, c);
            }
        }
        lane_reduce<COMP>(s, c, R);
        if (active && sub == 0) C.put(o, st_cvt<TOUT>(COMP ? s + c : s));
        oh += oq;
        ol += orr;
        if (ol >= n_olo) {
            ol -= n_olo;
            ++oh;
        }
    }
}

// C offsets of indices x[] of a label group from its digit descriptors (per
// label, last fastest: extent, magic (2 words), stride; from word w0 on).
// The descriptors are wave-uniform, so a digit costs a lane read per word
// and a few vector operations per index, all indices side by side.
// narrow: x, extents <= 4096 and C below 2^24 elements: 24-bit products (full
// rate; 32-bit ones run at a quarter of it).  The magic rounded to 24 bits
// exceeds 2^24 / d by less than 1.0001, exact while x d < 2^24 / 1.0001.
template <int NV>
__device__ __forceinline__ void digit_offsets(const StepWords &p, int w0, int nl, bool narrow, uint32_t (&x)[NV],
                                              int (&off)[NV]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) off[v] = 0;
    if (nl == 0) return;
    if (narrow) {
        for (int w = w0 + 4 * (nl - 1); w > w0; w -= 4) {
            const uint32_t ext = (uint32_t)p.digit(w);
            const uint32_t m24 = (((uint32_t)p.digit(w + 2) << 16) | ((uint32_t)p.digit(w + 1) >> 16)) + 1u;
            const uint32_t stride = (uint32_t)p.digit(w + 3);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const uint32_t xs = (x[v] << 8) & 0xffffffu;
                const uint32_t quo = (uint32_t)(((uint64_t)xs * (m24 & 0xffffffu)) >> 32);
                off[v] += (int)__umul24(x[v] - __umul24(quo, ext), stride);
                x[v] = quo;
            }
        }
        const uint32_t stride = (uint32_t)p.digit(w0 + 3);  // the slowest digit is what is left
#pragma unroll
        for (int v = 0; v < NV; ++v) off[v] += (int)__umul24(x[v], stride);
    } else {
        for (int w = w0 + 4 * (nl - 1); w > w0; w -= 4) {
            const uint32_t ext = (uint32_t)p.digit(w);
            const uint64_t magic = ((uint64_t)(uint32_t)p.digit(w + 2) << 32) | (uint32_t)p.digit(w + 1);
            const int stride = p.digit(w + 3);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const uint32_t quo = (uint32_t)(((uint64_t)x[v] * magic) >> 40);
                off[v] += (int)(x[v] - quo * ext) * stride;
                x[v] = quo;
            }
        }
        const int stride = p.digit(w0 + 3);
#pragma unroll
        for (int v = 0; v < NV; ++v) off[v] += (int)x[v] * stride;
    }
}
__device__ __forceinline__ bool narrow_digits(int M, int N) { return M <= 4080 && N <= 4080 && M * N < (1 << 24); }

// Register-tiled step: C[tcm[m] + tcn[n]] = sum_k A[k*M + m] * B[k*N + n].
// Thread (tx, ty) of a GX x (kBlk/GX) grid owns outputs m = m0 + tx + GX*i,
// n = n0 + ty + GY*j (i < TM, j < TN).  Across a wave, A reads are
// consecutive or broadcast, B reads broadcast or consecutive.
template <typename T, typename ACC, int TM, int TN, typename TOUT, typename P>
__device__ __forceinline__ void tstep(P A, P B, const Dest<TOUT> &C, const StepWords &p, const int tid,
                                      const int nthr) {
    const int M = p(4), N = p(5), K = p(6), GX = p(9), nm = p(11), nn_l = p(12);
    const int lgx = 31 - __clz(GX);
    const int GY = nthr >> lgx;
    const int tx = tid & (GX - 1), ty = tid >> lgx;
    const int SM = GX * TM, SN = GY * TN;
    for (int m0 = 0; m0 < M; m0 += SM) {
        if (m0 + tx >= M) break;
        for (int n0 = 0; n0 < N; n0 += SN) {
            if (n0 + ty >= N) break;
            int mi[TM], nj[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int m = m0 + tx + GX * i;
                mi[i] = m < M ? m : M - 1;
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int nn = n0 + ty + GY * j;
                nj[j] = nn < N ? nn : N - 1;
            }
            // U independent partial sums over k hide LDS latency (ILP)
            constexpr int U = TM * TN >= 16 ? 1 : (TM * TN >= 8 ? 2 : (TM * TN >= 4 ? 4 : 8));
            ACC acc[U][TM][TN];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[u][i][j] = 0;
            P a = A, b = B;
            int k = 0;
            for (; k + U <= K; k += U) {
                T av[U][TM], bv[U][TN];
#pragma unroll
                for (int u = 0; u < U; ++u) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) av[u][i] = a[u * M + mi[i]];
#pragma unroll
                    for (int j = 0; j < TN; ++j) bv[u][j] = b[u * N + nj[j]];
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[u][i][j] += (ACC)av[u][i] * (ACC)bv[u][j];
                a += U * M;
                b += U * N;
            }
            for (; k < K; ++k) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[0][i][j] += (ACC)a[mi[i]] * (ACC)b[nj[j]];
                a += M;
                b += N;
            }
#pragma unroll
            for (int u = 1; u < U; ++u)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[0][i][j] += acc[u][i][j];
            uint32_t xn[TN], xm[TM];
            int cn[TN], cm[TM];
#pragma unroll
            for (int j = 0; j < TN; ++j) xn[j] = (uint32_t)nj[j];
#pragma unroll
            for (int i = 0; i < TM; ++i) xm[i] = (uint32_t)mi[i];
            digit_offsets<TN>(p, 4 * nm, nn_l, narrow_digits(M, N), xn, cn);
            digit_offsets<TM>(p, 0, nm, narrow_digits(M, N), xm, cm);
#pragma unroll
            for (int i = 0; i < TM; ++i)
                if (m0 + tx + GX * i < M) {
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        if (n0 + ty + GY * j < N) C.put(cm[i] + cn[j], st_cvt<TOUT>(acc[0][i][j]));
                }
        }
    }
}

// Matrix-core tiled step (same contract as tstep): 16x16 output blocks,
// one wave per block, K in slices of 4 through the FP64 or FP32 16x16x4
// MFMA with accumulation in the compute type.  Lane l supplies
// A(m = 16 bm + l % 16, k = k0 + l / 16) and B(n = 16 bn + l % 16, same k)
// (zero outside the matrices) and receives column l % 16 of the block in
// rows FMfma<T>::row(l, r), r = 0..3.
template <typename T>
struct FMfma;
template <>
struct FMfma<double> {
    typedef double acc __attribute__((ext_vector_type(4)));
    __device__ __forceinline__ static acc mma(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    __device__ __forceinline__ static int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <>
struct FMfma<float> {
    typedef float acc __attribute__((ext_vector_type(4)));
    __device__ __forceinline__ static acc mma(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ __forceinline__ static int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// Products of the BM x BN blocks from (bm, bn) on over K summed terms from A
// and B on.  The blocks share their operands' reads, and 16 values of K are
// read while the previous 16 are multiplied: operands outside LDS arrive at the
// rate of the L1 cache (64 bytes a clock, which single blocks use up) instead
// of one round trip per 16.  A 144 x 144 x 216 step with both operands outside
// took 262 000 cycles with single blocks and no read ahead.
// 32 terms are summed by the matrix core before they join the result's running
// sum: chains of additions K long lose more than the partial sums of the
// register tiles and of lanes that share a sum.  Relative error of 1024
// 64-vertex rings, geometric mean, FP64 and FP32: register tiles and shared sums
// only 1.48e-15, 8.5e-7; here with two chains of K / 2 terms 1.72e-15, 9.3e-7,
// joined every 32 terms 1.41e-15, 7.9e-7, every 16 1.32e-15, 7.8e-7.  Batches of
// 60 BF16 and 256 FP64 rings, 1024 grids: two chains 447, 1042, 134 us; joined
// every 32 terms 452, 1050, 133; every 16 453, 1056, 133; as two half sums every
// 32 (whose registers cost the grids 1 to 2 %) 456, 1058, 135 at 1.27e-15, 7.3e-7.
template <int BM, int BN, typename T, typename P>
__device__ __forceinline__ void mblock(P A, P B, const int M, const int N, const int K, const int bm, const int bn,
                                       const int lane, typename FMfma<T>::acc (&acc)[BM][BN]) {
    typedef FMfma<T> Op;
    typedef typename Op::acc Acc;
    const int li = lane & 15, lk = lane >> 4;
    int am[BM], bx[BN];  // operand columns (0 outside the matrix: mok and nok are false there, products zero)
    bool mok[BM], nok[BN];
#pragma unroll
    for (int i = 0; i < BM; ++i) {
        const int m = (bm * BM + i) * 16 + li;
        mok[i] = m < M;
        am[i] = mok[i] ? m : 0;
    }
#pragma unroll
    for (int j = 0; j < BN; ++j) {
        const int n = (bn * BN + j) * 16 + li;
        nok[j] = n < N;
        bx[j] = nok[j] ? n : 0;
    }
    Acc part[BM][BN];
    auto clear = [&] {
#pragma unroll
        for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int j = 0; j < BN; ++j) part[i][j] = Acc{0, 0, 0, 0};
    };
    auto join = [&] {
#pragma unroll
        for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int j = 0; j < BN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] += part[i][j][r];
    };
    auto mma_all = [&](T (&av)[BM], T (&bv)[BN], bool ok) {
        T a[BM], b[BN];
#pragma unroll
        for (int i = 0; i < BM; ++i) a[i] = mok[i] && ok ? av[i] : T(0);
#pragma unroll
        for (int j = 0; j < BN; ++j) b[j] = nok[j] && ok ? bv[j] : T(0);
#pragma unroll
        for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int j = 0; j < BN; ++j) part[i][j] = Op::mma(a[i], b[j], part[i][j]);
    };
    T av[4][BM], bv[4][BN];
    int ao = lk * M, bo = lk * N;
    auto load = [&](int u, int so, int to) {
#pragma unroll
        for (int i = 0; i < BM; ++i) av[u][i] = A[so + am[i]];
#pragma unroll
        for (int j = 0; j < BN; ++j) bv[u][j] = B[to + bx[j]];
    };
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) acc[i][j] = Acc{0, 0, 0, 0};
    clear();
    constexpr int kJoin = 2;
    int k = K, chunks = 0;
    if (k >= 16) {
#pragma unroll
        for (int u = 0; u < 4; ++u) load(u, ao + 4 * u * M, bo + 4 * u * N);
        for (;;) {
            T ac[4][BM], bc[4][BN];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int i = 0; i < BM; ++i) ac[u][i] = av[u][i];
#pragma unroll
                for (int j = 0; j < BN; ++j) bc[u][j] = bv[u][j];
            }
            k -= 16;
            ao += 16 * M;
            bo += 16 * N;
            if (k >= 16) {
#pragma unroll
                for (int u = 0; u < 4; ++u) load(u, ao + 4 * u * M, bo + 4 * u * N);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u) mma_all(ac[u], bc[u], true);
            if (k < 16) break;
            if (++chunks == kJoin) {
                join();
                clear();
                chunks = 0;
            }
        }
    }
    // the last k < 16: a pair of slices, then up to two
    const bool pair = k >= 8;
    const int rest = k & 7;
    if (pair) {
        load(0, ao, bo);
        load(1, ao + 4 * M, bo + 4 * N);
        ao += 8 * M;
        bo += 8 * N;
    }
    const bool ok0 = lk < rest, ok1 = lk + 4 < rest;
    if (rest > 0) load(2, ok0 ? ao : 0, ok0 ? bo : 0);
    if (rest > 4) load(3, ok1 ? ao + 4 * M : 0, ok1 ? bo + 4 * N : 0);
    if (pair) {
        mma_all(av[0], bv[0], true);
        mma_all(av[1], bv[1], true);
    }
    if (rest > 0) mma_all(av[2], bv[2], ok0);
    if (rest > 4) mma_all(av[3], bv[3], ok1);
    join();
}

// The blocks' results into C.
template <int BM, int BN, typename T, typename TOUT>
__device__ __forceinline__ void mstore(const Dest<TOUT> &C, const StepWords &p, const int bm, const int bn,
                                       const int lane, const typename FMfma<T>::acc (&acc)[BM][BN]) {
    typedef FMfma<T> Op;
    const int M = p(4), N = p(5), nm = p(11), nn_l = p(12), li = lane & 15;
    const bool narrow = narrow_digits(M, N);
    bool nok[BN];
    uint32_t xn[BN];
    int cn[BN];
#pragma unroll
    for (int j = 0; j < BN; ++j) {
        const int n = (bn * BN + j) * 16 + li;
        nok[j] = n < N;
        xn[j] = (uint32_t)n;
    }
    digit_offsets<BN>(p, 4 * nm, nn_l, narrow, xn, cn);
#pragma unroll
    for (int i = 0; i < BM; ++i) {
        const int m0 = (bm * BM + i) * 16;
        uint32_t xm[4];
        int cm[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) xm[r] = (uint32_t)(m0 + Op::row(lane, r));
        digit_offsets<4>(p, 0, nm, narrow, xm, cm);
        if (C.in_lds) {
#pragma unroll
            for (int j = 0; j < BN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (nok[j] && m0 + Op::row(lane, r) < M) C.l[cm[r] + cn[j]] = st_cvt<TOUT>(acc[i][j][r]);
        } else {
#pragma unroll
            for (int j = 0; j < BN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (nok[j] && m0 + Op::row(lane, r) < M) C.g[cm[r] + cn[j]] = st_cvt<TOUT>(acc[i][j][r]);
        }
    }
}

template <int BM, int BN, typename T, typename TOUT, typename P>
__device__ __forceinline__ void mstep(P A, P B, const Dest<TOUT> &C, const StepWords &p, const int tid, const int nthr) {
    const int M = p(4), N = p(5), K = p(6);
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nbm = (M + 16 * BM - 1) / (16 * BM), nbn = (N + 16 * BN - 1) / (16 * BN);
    const int nw = nthr >> 6;
    int bm = 0, bn = wave;  // block bm * nbn + bn, advanced without divisions
    while (bn >= nbn) {
        bn -= nbn;
        ++bm;
    }
    while (bm < nbm) {
        typename FMfma<T>::acc acc[BM][BN];
        mblock<BM, BN, T>(A, B, M, N, K, bm, bn, lane, acc);
        mstore<BM, BN, T>(C, p, bm, bn, lane, acc);
        bn += nw;
        while (bn >= nbn) {
            bn -= nbn;
            ++bm;
        }
    }
}

// A step of few blocks and a long sum that has all of the workgroup's waves
// (planned only alone in its phase): p(8) ranges of K, each block of a range a
// wave; the first range's waves add the others' results, in order, from LDS
// (element p(9) on, 256 values a block).  One wave per block took 24 outputs
// of 3456 terms, operands outside LDS, 150 000 cycles, and lanes that share an
// output's sum 162 000.
template <typename T, typename TOUT, typename P>
__device__ __forceinline__ void msplit(P A, P B, const Dest<TOUT> &C, const StepWords &p, T *sm, const int tid) {
    const int M = p(4), N = p(5), K = p(6), parts = p(8);
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nbm = (M + 15) >> 4, nbn = (N + 15) >> 4, nb = nbm * nbn;
    int part = 0, blk = wave;
    while (blk >= nb) {
        blk -= nb;
        ++part;
    }
    int bm = 0, bn = blk;
    while (bn >= nbn) {
        bn -= nbn;
        ++bm;
    }
    const int kper = ((K + parts - 1) / parts + 3) & ~3;
    const int k0 = part * kper, kn = part < parts ? min(K - k0, kper) : 0;
    LdsPtr<T> red = (LdsPtr<T>)(sm + p(9));
    typename FMfma<T>::acc acc[1][1];
    if (part < parts) {
        if (kn > 0)
            mblock<1, 1, T>(A + k0 * M, B + k0 * N, M, N, kn, bm, bn, lane, acc);
        else
            acc[0][0] = typename FMfma<T>::acc{0, 0, 0, 0};
        if (part > 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) red[((part - 1) * nb + blk) * 256 + 64 * r + lane] = acc[0][0][r];
        }
    }
    __syncthreads();
    if (part == 0) {
        for (int q = 1; q < parts; ++q) {
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[0][0][r] += red[((q - 1) * nb + blk) * 256 + 64 * r + lane];
        }
        mstore<1, 1, T>(C, p, bm, bn, lane, acc);
    }
}

template <typename T, typename ACC, typename TOUT, typename P>
__device__ __forceinline__ void tstep_sel(P A, P B, const Dest<TOUT> &C, const StepWords &p, T *sm,
                                          const int tid, const int nthr) {
    const int TM = p(7), TN = p(8);
    if constexpr (std::is_same<T, ACC>::value) {
        if (TM == 0) {  // matrix-core mode
            // four blocks a wave where every wave has that many
            if (((p(4) + 31) >> 5) * ((p(5) + 31) >> 5) >= (nthr >> 6))
                mstep<2, 2, T>(A, B, C, p, tid, nthr);
            else
                mstep<1, 1, T>(A, B, C, p, tid, nthr);
            return;
        }
        if (TM < 0) {
            msplit<T>(A, B, C, p, sm, tid);
            return;
        }
    }
    switch (TM * 8 + TN) {
        case 9: tstep<T, ACC, 1, 1>(A, B, C, p, tid, nthr); break;
        case 10: tstep<T, ACC, 1, 2>(A, B, C, p, tid, nthr); break;
        case 12: tstep<T, ACC, 1, 4>(A, B, C, p, tid, nthr); break;
        case 17: tstep<T, ACC, 2, 1>(A, B, C, p, tid, nthr); break;
        case 18: tstep<T, ACC, 2, 2>(A, B, C, p, tid, nthr); break;
        case 20: tstep<T, ACC, 2, 4>(A, B, C, p, tid, nthr); break;
        case 33: tstep<T, ACC, 4, 1>(A, B, C, p, tid, nthr); break;
        case 34: tstep<T, ACC, 4, 2>(A, B, C, p, tid, nthr); break;
        default: tstep<T, ACC, 4, 4>(A, B, C, p, tid, nthr); break;
    }
}

// One step on its waves (threads tid of nthr).
//   OP_TSTEP: [a, b, c, M, N, K, TM, TN, GX, final, nm, nn, w0, nw, digits of M, digits of N]
//             (TM = 0: matrix-core mode, planned only where the accumulator is
//             the compute type; TM = -1: the same with K split into TN ranges,
//             GX the LDS element offset of their sums)
//   OP_STEP:  [a, b, c, n_ohi, n_olo, n_shi, n_slo, t_ohi, t_olo, t_shi, t_slo, R, final, slot, w0, nw]
// Operands in LDS take a body of their own (LDS reads, not flat ones).
template <int BLK, typename T, int FM>
__device__ __forceinline__ void run_step(const StepWords &p, T *sm, T *scr, void *out, const int32_t *slots,
                                         int slot_words, unsigned char *red) {
    typedef typename std::conditional<FM == FM_INTER, T, double>::type TO;
    constexpr bool CMP = (FM == FM_COMP);
    const bool tiled = p(0) == OP_TSTEP;
    const int la = p(1), lb = p(2), lc = p(3);
    const int w0 = tiled ? p(13) : p(15), nw = tiled ? p(14) : p(16);
    const bool fin = (tiled ? p(10) : p(13)) != 0;
    const int tid = threadIdx.x - 64 * w0, nthr = 64 * nw;
    const bool unary = !tiled && lb == -1;
    const bool in_lds = la >= 0 && (unary || lb >= 0);
    const int2 *tab = reinterpret_cast<const int2 *>(slots + (tiled ? 0 : p(14) * slot_words));
    Dest<T> C;
    C.in_lds = !fin && lc >= 0;
    C.l = (LdsPtr<T>)(sm + (C.in_lds ? lc : 0));
    C.g = (GlobalPtr<T>)(fin ? (T *)out : scr + (lc < 0 ? -lc - 2 : 0));
    auto go = [&](auto A, auto B) {
        if (FM == FM_INTER || !fin) {
            if (tiled)
                tstep_sel<T, T>(A, B, C, p, sm, tid, nthr);
            else if (unary)
                fstep<BLK, T, false, true>(A, B, C, tab, p, (T *)red, tid, nthr);
            else
                fstep<BLK, T, false, false>(A, B, C, tab, p, (T *)red, tid, nthr);
        } else {
            const Dest<TO> O = {false, nullptr, (GlobalPtr<TO>)out};
            if (tiled)
                tstep_sel<T, TO>(A, B, O, p, sm, tid, nthr);
            else if (unary)
                fstep<BLK, TO, CMP, true>(A, B, O, tab, p, (TO *)red, tid, nthr);
            else
                fstep<BLK, TO, CMP, false>(A, B, O, tab, p, (TO *)red, tid, nthr);
        }
    };
    if (in_lds) {
        go((LdsPtr<const T>)(sm + la), (LdsPtr<const T>)(sm + (unary ? 0 : lb)));
    } else {
        const T *A = la >= 0 ? sm + la : scr + (-la - 2);
        const T *B = unary ? A : (lb >= 0 ? sm + lb : scr + (-lb - 2));
        go(A, B);
    }
}

// The copies of one phase: n ops [kind (0: image tables, 1: workspace), src
// chunk, chunks, dst chunk] of five words (the first is the opcode), word i in
// lane i of r.  16-byte chunks go from global memory straight to LDS (no
// registers, nothing to wait for until the phase ends), 64 consecutive
// chunks an instruction.  Ops of up to 64 chunks go to the waves in turn,
// larger ones are shared by all.
constexpr int kCopyBatch = 12;  // ops in 64 words
template <int BLK>
__device__ __forceinline__ void issue_copies(int32_t r, int first, int n, const int32_t *tabs, const void *scratch,
                                             unsigned char *lds, int lane, int wave) {
    typedef __attribute__((address_space(1))) const uint32_t g_word;
    typedef __attribute__((address_space(3))) uint32_t l_word;
    constexpr int W = BLK / 64;
    for (int i = 0; i < n; ++i) {
        const int w = first + 5 * i, chunks = __builtin_amdgcn_readlane(r, w + 3);
        const int seg = (wave - i) & (W - 1);
        if (64 * seg >= chunks) continue;
        const int kind = __builtin_amdgcn_readlane(r, w + 1), src = __builtin_amdgcn_readlane(r, w + 2);
        const int dst = __builtin_amdgcn_readlane(r, w + 4);
        const unsigned char *from =
            (kind == 0 ? (const unsigned char *)tabs : (const unsigned char *)scratch) + 16 * (int64_t)src;
        for (int c0 = 64 * seg; c0 < chunks; c0 += BLK)
            if (c0 + lane < chunks)
                __builtin_amdgcn_global_load_lds((g_word *)(from + 16 * (c0 + lane)), (l_word *)(lds + 16 * (dst + c0)),
                                                 16, 0, 0);
    }
}

// Waits for the wave's global loads (also those on their way to LDS).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }

// The fused kernel: one network per workgroup.  The program's index (words
// from header word 2 on: the number of phases, then per phase the word
// offset and number of its copies and, per wave, the word offset of its
// step or 0) leads every wave straight to its own work.  A phase issues the
// copies for the next one (regions no step of the phase touches), runs
// its steps (each on its own waves), waits for the copies and ends with a
// barrier.
template <int BLK, typename T, typename TIN, int FM>
__device__ __forceinline__ void fused_body(const FusedDesc &d, void *const *__restrict__ outs,
                                           int64_t *__restrict__ stamps, void *out1,
                                           int64_t *__restrict__ phase_ticks, int max_phases, int64_t t0) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int W = BLK / 64, S = 2 + W;  // waves; index words per phase
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int net = d.net, n_words = d.n_words;
    const int32_t *img = reinterpret_cast<const int32_t *>(smem);
    // header and the first ops: phase 0 (copies only) starts from them while
    // the program is on its way to LDS
    int32_t head = lane < n_words ? d.prog[lane] : 0;
    {
        // the program itself is one copy (words a multiple of four)
        typedef __attribute__((address_space(1))) const uint32_t g_word;
        typedef __attribute__((address_space(3))) uint32_t l_word;
        for (int c0 = 64 * wave; c0 < n_words / 4; c0 += BLK)
            if (c0 + lane < n_words / 4)
                __builtin_amdgcn_global_load_lds((g_word *)(d.prog + 4 * (c0 + lane)), (l_word *)(smem + 16 * c0), 16,
                                                 0, 0);
    }
    if (d.n_fprep > 0) {
        // materialise the network's (few) inputs into its workspace, one wave
        // per entry, then make the writes visible to the workgroup's reads
        for (int j = wave; j < d.n_fprep; j += W) fprep_tiny<T, TIN>(d.fprep[j], lane);
        __threadfence();
        __syncthreads();
    }
    const int slot0 = __builtin_amdgcn_readlane(head, 3), slot_words = __builtin_amdgcn_readlane(head, 4);
    const int index = __builtin_amdgcn_readlane(head, 2);
    unsigned char *red = smem + __builtin_amdgcn_readlane(head, 5);  // reduction scratch (256 bytes)
    const int32_t *slots = img + slot0;
    const int32_t *tabs = d.prog + __builtin_amdgcn_readlane(head, 6);
    T *sm = reinterpret_cast<T *>(smem);
    T *scr = (T *)d.scratch;
    void *out = out1 ? out1 : outs[net];
    int n_copies = 0;  // of phase 0, among the first 64 words
    while (8 + 5 * n_copies + 4 < 64 && __builtin_amdgcn_readlane(head, 8 + 5 * n_copies) == OP_COPY) ++n_copies;
    issue_copies<BLK>(head, 8, n_copies, tabs, d.scratch, smem, lane, wave);
    wait_loads();
    __syncthreads();
    const int32_t *const entries = index < n_words ? img : d.prog;  // the index, in LDS where it fits
    const int n_phases = __builtin_amdgcn_readfirstlane(entries[index]);
    int at = index + 1;
    int32_t ix = lane < S ? entries[at + lane] : 0;
    for (int phase = 0; phase < n_phases; ++phase) {
        const int c_off = __builtin_amdgcn_readlane(ix, 0), c_n = __builtin_amdgcn_readlane(ix, 1);
        const int step = __builtin_amdgcn_readlane(ix, 2 + wave);
        if (phase > 0 || c_n > n_copies) {
            const int done = phase > 0 ? 0 : n_copies;
            for (int i = done; i < c_n; i += kCopyBatch) {
                const int o = c_off + 5 * i;
                const int32_t r = o + lane < n_words ? img[o + lane] : 0;
                issue_copies<BLK>(r, 0, min(kCopyBatch, c_n - i), tabs, d.scratch, smem, lane, wave);
            }
        }
        const StepWords p(img, n_words, step, lane);
        at += S;
        ix = lane < S && phase + 1 < n_phases ? entries[at + lane] : 0;  // the next phase's
        if (step) run_step<BLK, T, FM>(p, sm, scr, out, slots, slot_words, red);
        wait_loads();
        if (phase > 0 || c_n > n_copies) __syncthreads();
        if (phase_ticks && threadIdx.x == 0 && phase < max_phases)
            phase_ticks[(int64_t)net * max_phases + phase] = (int64_t)wall_clock64();
    }
    if (stamps && threadIdx.x == 0) {
        stamps[2 * net] = t0;
        stamps[2 * net + 1] = (int64_t)wall_clock64();
    }
}

template <int BLK, typename T, typename TIN, int FM>
__global__ __launch_bounds__(BLK) __attribute__((amdgpu_waves_per_eu(2))) void k_fused(
    const FusedDesc *__restrict__ nets, void *const *__restrict__ outs, int64_t *__restrict__ stamps, void *out1,
    int64_t *__restrict__ phase_ticks, int max_phases) {
    const int64_t t0 = stamps ? (int64_t)wall_clock64() : 0;
    const FusedDesc d = nets[blockIdx.x];
    fused_body<BLK, T, TIN, FM>(d, outs, stamps, out1, phase_ticks, max_phases, t0);
}

template <int BLK, typename T, typename TIN, int FM>
static hipError_t go_fused(const FusedDesc *nets, void *const *outs, int64_t *stamps,
                           void *out1, int64_t *phase_ticks, int max_phases, int n_blocks, int lds_bytes,
                           hipStream_t st) {
    static int configured = -1;
    if (lds_bytes > configured) {
        hipError_t e = hipFuncSetAttribute((const void *)k_fused<BLK, T, TIN, FM>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
        configured = lds_bytes;
    }
    hipLaunchKernelGGL((k_fused<BLK, T, TIN, FM>), dim3(n_blocks), dim3(BLK), lds_bytes, st, nets, outs,
                       stamps, out1, phase_ticks, max_phases);
    return hipGetLastError();
}

template <int BLK>
hipError_t launch_fused_blk(const FusedDesc *nets, void *const *outs, int64_t *stamps,
                            void *out1, int64_t *phase_ticks, int max_phases, int n_blocks, int lds_bytes, int compute,
                            int fm, hipStream_t st) {
#define HTN_GO(T, TIN, F) go_fused<BLK, T, TIN, F>(nets, outs, stamps, out1, phase_ticks, max_phases, n_blocks, lds_bytes, st)
    if (compute == 0) return fm == FM_COMP ? HTN_GO(double, double, FM_COMP) : HTN_GO(double, double, FM_INTER);
    if (compute == 1) {
        if (fm == FM_COMP) return HTN_GO(float, float, FM_COMP);
        if (fm == FM_F64) return HTN_GO(float, float, FM_F64);
        return HTN_GO(float, float, FM_INTER);
    }
    if (compute == 2) {
        if (fm == FM_COMP) return HTN_GO(float, bf16_t, FM_COMP);
        if (fm == FM_F64) return HTN_GO(float, bf16_t, FM_F64);
        return HTN_GO(float, bf16_t, FM_INTER);
    }
#undef HTN_GO
    return hipErrorInvalidValue;
}

}  // namespace kern
}  // namespace htn
