// Device bodies shared by the per-step kernels (kernels.hip) and the
// persistent work queue (queue.hip), so that a step gives the same result
// bit for bit whichever of the two runs it.
#pragma once

#include "kern_common.hpp"

namespace htn {
namespace kern {

// NB terms of one lane's share of an output's sum from (sh, sl) on, added in
// order; all of them are read before the first is added.
template <int NB, typename TA, typename TB, typename ACC, bool UNARY, bool COMP>
__device__ __forceinline__ void add_terms(const TA *a0, const TB *b0, const int2 *__restrict__ th,
                                          const int2 *__restrict__ tl, int &sh, int &sl, int dq, int dr, int n_slo,
                                          ACC &acc, ACC &cmp) {
    int2 h[NB], l[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        h[u] = th[sh];
        l[u] = tl[sl];
        sh += dq;
        sl += dr;
        if (sl >= n_slo) {
            sl -= n_slo;
            ++sh;
        }
    }
    ACC pv[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        pv[u] = Ld<ACC, TA>::get(a0 + h[u].x + l[u].x);
        if constexpr (!UNARY) pv[u] *= Ld<ACC, TB>::get(b0 + h[u].y + l[u].y);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) accum<COMP>(acc, cmp, pv[u]);
}

// One lane's share of an output's sum: terms (sh, sl), (sh, sl) + stride, ...
// (stride = dq * n_slo + dr, dr < n_slo), `count` of them, added in that
// order.  Each term is a chain of loads (two table entries, then the operands
// they address, a microsecond or two end to end), so terms are read eight
// (then four, two, one) ahead of their additions: the final sum of a
// 124 416-term network (60 groups of 64 lanes, 33 terms a lane) 18.8 -> 8.3 us.
template <typename TA, typename TB, typename ACC, bool UNARY, bool COMP>
__device__ __forceinline__ void lane_terms(const TA *a0, const TB *b0, const int2 *__restrict__ th,
                                           const int2 *__restrict__ tl, int sh, int sl, int dq, int dr, int n_slo,
                                           int64_t count, ACC &acc, ACC &cmp) {
    for (; count >= 8; count -= 8)
        add_terms<8, TA, TB, ACC, UNARY, COMP>(a0, b0, th, tl, sh, sl, dq, dr, n_slo, acc, cmp);
    if (count & 4) add_terms<4, TA, TB, ACC, UNARY, COMP>(a0, b0, th, tl, sh, sl, dq, dr, n_slo, acc, cmp);
    if (count & 2) add_terms<2, TA, TB, ACC, UNARY, COMP>(a0, b0, th, tl, sh, sl, dq, dr, n_slo, acc, cmp);
    if (count & 1) add_terms<1, TA, TB, ACC, UNARY, COMP>(a0, b0, th, tl, sh, sl, dq, dr, n_slo, acc, cmp);
}

// Block `blk` of the pairwise step C[o] = sum_s A[.]*B[.] (k_step's grid:
// R lanes per output, outputs in block order; with split sums, `split`
// lane groups per output write (sum, compensation) partials).
template <typename TA, typename TB, typename TC, typename ACC, bool UNARY, bool COMP>
__device__ __forceinline__ void step_block(const TA *__restrict__ A, const TB *__restrict__ B, TC *__restrict__ C,
                                           const int2 *__restrict__ tab, const StepArgs &s, int64_t blk) {
    const int64_t gt = blk * kBlk + threadIdx.x;
    const int64_t grp = gt >> s.log2R;
    const int64_t o = s.split > 1 ? grp / s.split : grp;
    const int jc = (int)(grp - o * s.split);  // chunk of the summed range (split > 1)
    const int sub = (int)(gt & (s.R - 1));
    const bool active = o < s.n_out;
    ACC acc = 0, cmp = 0;
    if (active) {
        const int oh = (int)(o / s.n_olo);
        const int ol = (int)(o - (int64_t)oh * s.n_olo);
        const int2 x = tab[s.t_ohi + oh], y = tab[s.t_olo + ol];
        const TA *a0 = A + (x.x + y.x);
        const TB *b0 = B;
        if constexpr (!UNARY) b0 = B + (x.y + y.y);
        // the lane's terms: sub, sub + R, ... of the (chunk of the) summed range
        const int64_t n_sum = (int64_t)s.n_shi * s.n_slo;
        int64_t e = sub, e_end = n_sum;
        if (s.split > 1) {
            e = (int64_t)jc * s.chunk + sub;
            e_end = min(n_sum, (int64_t)(jc + 1) * s.chunk);
        }
        const int dq = s.R / s.n_slo, dr = s.R - dq * s.n_slo;
        if (!UNARY && s.R == 1 && s.split <= 1) {
            // every lane of the wave reads the same table entries: scalar loads
            // (per lane 2500 x 2501 sums of 256 FP32 terms took 1803 us, not 649)
            lane_terms<TA, TB, ACC, UNARY, COMP>(a0, b0, tab + s.t_shi, tab + s.t_slo, 0, 0, dq, dr, s.n_slo, n_sum,
                                                 acc, cmp);
        } else if (e < e_end) {
            const int sh = (int)(e / s.n_slo), sl = (int)(e - (int64_t)sh * s.n_slo);
            lane_terms<TA, TB, ACC, UNARY, COMP>(a0, b0, tab + s.t_shi, tab + s.t_slo, sh, sl, dq, dr, s.n_slo,
                                                 (e_end - e + s.R - 1) >> s.log2R, acc, cmp);
        }
    }
    lane_reduce<COMP>(acc, cmp, s.R);
    if (active && sub == 0) {
        if (s.split > 1) {
            double *q = s.part + 2 * (o * s.split + jc);
            q[0] = (double)acc;
            q[1] = COMP ? (double)cmp : 0.0;
        } else {
            C[o] = st_cvt<TC>(COMP ? acc + cmp : acc);
        }
    }
}

// Second pass of a split sum for output o, run by one wave (lane = lane
// index): lanes stride over the `split` partial (sum, compensation) pairs,
// then a fixed shuffle tree combines them.
template <typename TC, bool COMP>
__device__ __forceinline__ void split_finish_one(const double *__restrict__ part, TC *__restrict__ C, int split,
                                                 int64_t o, int lane) {
    double sum = 0.0, cmp = 0.0;
    for (int j = lane; j < split; j += 64) {
        const double *q = part + 2 * (o * split + j);
        combine<COMP>(sum, cmp, q[0], q[1]);
    }
    lane_reduce<COMP>(sum, cmp, 64);
    if (lane == 0) C[o] = st_cvt<TC>(COMP ? sum + cmp : sum);
}

__device__ __forceinline__ int prep_div(int e, uint32_t mul, int sh) {
    return (int)(__umulhi((uint32_t)e << 1, mul) >> sh);
}

// Elements e0, e0 + step, ... (NB of them) of a scaled-input
// materialisation: the input entry (through the source gather table when the
// layout changes) times each folded coefficient tensor's entry, in the
// intermediate type.  The NB elements are independent chains of loads side
// by side, and quotients come from a multiplication: a division of an int
// is some forty instructions, and with one per table look-up they, not
// memory, set the time.
template <int NB, typename TIN, typename TI>
__device__ __forceinline__ void prep_values(const PrepDesc &q, const int2 *__restrict__ tab, int e0, int step,
                                            TI (&v)[NB]) {
    const TIN *src = (const TIN *)q.src;
    int se[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) se[u] = e0 + u * step;
    if (q.snlo > 0) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int e = se[u], eh = prep_div(e, q.smul, q.ssh);
            se[u] = tab[q.sthi + eh].x + tab[q.stlo + (e - eh * q.snlo)].x;
        }
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) v[u] = Ld<TI, TIN>::get(src + se[u]);
    for (int k = 0; k < q.ns; ++k) {
        TI c[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int e = e0 + u * step, eh = prep_div(e, q.mul[k], q.sh[k]);
            c[u] = Ld<TI, TIN>::get((const TIN *)q.sp[k] + tab[q.thi[k] + eh].x +
                                    tab[q.tlo[k] + (e - eh * q.nlo[k])].x);
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) v[u] *= c[u];
    }
}

// Elements first, first + step, ... below end, four at a time.
template <typename TIN, typename TI>
__device__ __forceinline__ void prep_range(const PrepDesc &q, const int2 *__restrict__ tab, TI *__restrict__ dst,
                                           int64_t first, int64_t end, int step) {
    int64_t e = first;
    for (; e + 3 * (int64_t)step < end; e += 4 * (int64_t)step) {
        TI v[4];
        prep_values<4, TIN, TI>(q, tab, (int)e, step, v);
#pragma unroll
        for (int u = 0; u < 4; ++u) dst[e + u * (int64_t)step] = v[u];
    }
    for (; e < end; e += step) {
        TI v[1];
        prep_values<1, TIN, TI>(q, tab, (int)e, step, v);
        dst[e] = v[0];
    }
}

}  // namespace kern
}  // namespace htn
