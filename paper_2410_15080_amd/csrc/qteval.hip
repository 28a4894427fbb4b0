// QT evaluator (Sec. 6.2): exact statevector simulation of subcircuit
// instances on the GPU, and the assembly of quantum-tensor entries as signed
// sums of instance results.
//
// Qubit q of an n-qubit instance is bit n-1-q of the amplitude index
// (qubit 0 slowest, as a row-major (2,)*n array).  The ops arrive as the
// schedule of sv_plan.cpp: a group names K amplitude bits, each thread takes
// the 2^K amplitudes that differ in them into registers, applies every op of
// the group there (unitaries on the K bits; CZ, RZZ, projections and
// controls on any bits) and puts them back into LDS, one barrier a group
// instead of one an op.  A workgroup reads its records in LDS, kRecChunk at a
// time: read where they lie, each new record costs a memory round trip.
//
// A state of up to kSvLdsQubits qubits lives in LDS from its preparation to
// its measurement (k_sv_small).  A larger one lies in device memory and
// is worked through in passes, one launch each, over tiles of kSvTileBits
// amplitude bits chosen per pass so that as many ops as possible run in it
// (k_sv_pass), and is measured from there (k_sv_measure); instances with
// the same preparation and ops share one state.
//
// What bounds it: the FP64 units for the large states, the latency of a few
// dozen dependent records for the small ones (a record took 0.4 us whatever
// it held until the CZ gates and unitaries of a group were packed into
// layers).  Two 15-qubit subcircuits of 4 layers (80 instances, 37 distinct
// states): evaluation and contraction 4 317 -> 86 us; the 44 instances of 3 to
// 5 qubits of the 10-qubit circuit 44.2 -> 19.4 us, contraction included.  Before,
// one workgroup per instance ran every op as a pass over its state.
//
// Unitaries merged on the host are rounded once for the whole state: their
// error of the norm is common to all amplitudes and does not average out of
// an output.  The host knows it (products in 80 bits) and puts it into the
// state's correction.  QT entries of those two workloads against 80-bit states,
// root mean square of four sets of angles: op by op 3.3e-16 and 6.0e-16, merged
// without the correction 5.9e-16 and 5.7e-16, with it 4.1e-16 and 5.0e-16; of
// 12- and 11-qubit subcircuits 3.6e-16, 6.0e-16 and 3.4e-16.
//
// The result of a Pauli observable O = (x)_q P_q with projectors on the
// kept qubits,
//     out[x] = Re sum_{s: kept bits of s = x} conj(psi[s ^ m]) c(s) psi[s],
// uses O|s> = c(s) |s ^ m>: m flips the X and Y qubits, and
// c(s) = i^{#Y} (-1)^{popcount(s & (Z|Y qubits))}.  Each output's terms are
// summed in a fixed order (deterministic results).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kern_common.hpp"
#include "kernels.hpp"
#include "sv_plan.hpp"

namespace htn {
namespace kern {

namespace {

constexpr int kRecChunk = 32;  // records staged in LDS at a time

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// LDS slot of tile-local amplitude i: the low four bits (16 amplitudes are
// one row of the banks) are folded with the higher ones, so a wave whose
// lanes differ in any four neighbouring bits touches every bank once.
__device__ __forceinline__ int sv_slot(int i) { return i ^ ((i >> 4) & 15) ^ ((i >> 8) & 15); }

struct SvTables {
    SvRecord recs[kRecChunk];
    double2 plo[64], phi[64];  // product-state factors of the low six and the higher tile bits
    double2 clo[64], chi[64];  // and their corrections (SvState::corr), summed
    int32_t dlo[64], dhi[64];  // amplitude index bits of the low six and the higher tile bits
};

__device__ __forceinline__ void load_recs(SvTables &T, const SvRecord *__restrict__ recs, int first, int n_rec,
                                          int threads) {
    constexpr int Q = sizeof(SvRecord) / 16;
    const int4 *src = reinterpret_cast<const int4 *>(recs + first);
    int4 *dst = reinterpret_cast<int4 *>(T.recs);
    const int m = min(kRecChunk, n_rec - first) * Q;
    for (int i = threadIdx.x; i < m; i += threads) dst[i] = src[i];
}

// Register r of a thread holds the amplitude whose group bits spell r.
template <int K, int B>
__device__ __forceinline__ void reg_u1(double2 (&v)[1 << K], const double *m) {
#pragma unroll
    for (int r = 0; r < (1 << K); ++r)
        if (!((r >> B) & 1)) {
            const double2 a = v[r], b = v[r | (1 << B)];
            v[r] = make_double2(fma(-m[3], b.y, fma(m[2], b.x, fma(-m[1], a.y, m[0] * a.x))),
                                fma(m[3], b.x, fma(m[2], b.y, fma(m[1], a.x, m[0] * a.y))));
            v[r | (1 << B)] = make_double2(fma(-m[7], b.y, fma(m[6], b.x, fma(-m[5], a.y, m[4] * a.x))),
                                           fma(m[7], b.x, fma(m[6], b.y, fma(m[5], a.x, m[4] * a.y))));
        }
}

// Conditions on amplitude bits split into the thread's (base) and the
// register's (dep[r], the same for every thread): the first is one vector
// comparison for all registers, the second is scalar.
template <int K, int B>
__device__ __forceinline__ void reg_cx(double2 (&v)[1 << K], int base, const int (&dep)[1 << K], int gmask,
                                       int control) {
    const bool on = (control & gmask) || (base & control);
#pragma unroll
    for (int r = 0; r < (1 << K); ++r)
        if (!((r >> B) & 1) && (!(control & gmask) || (dep[r] & control))) {
            const double2 a = v[r], b = v[r | (1 << B)];
            v[r] = on ? b : a;
            v[r | (1 << B)] = on ? a : b;
        }
}

__device__ __forceinline__ double flip(double x, uint32_t sign) {
    return __hiloint2double((int)((uint32_t)__double2hiint(x) ^ sign), __double2loint(x));
}

// Runs n_rec records on the 2^tb amplitudes of the tile in LDS; hi: the
// tile's own amplitude bits.  T.dlo / T.dhi are filled and the tile is in
// place (barrier passed); ends with a barrier.
template <int K, int THREADS>
__device__ __forceinline__ void run_records(double2 *st, SvTables &T, const SvRecord *__restrict__ recs, int n_rec,
                                            int tb, int hi) {
    constexpr int R = 1 << K;
    const bool active = (int)threadIdx.x < (1 << (tb - K));
    const bool idle = (int)(threadIdx.x & ~63u) >= (1 << (tb - K));  // wave-uniform: barriers only
    double2 v[R];
    int dep[R];                    // amplitude bits of register r
    int slot = 0, sx[K];           // LDS slot of register 0; what each group bit adds (slots are linear)
    int base = 0, gmask = 0;       // amplitude bits of the thread; of the group
#pragma unroll
    for (int r = 0; r < R; ++r) {
        v[r] = make_double2(0.0, 0.0);
        dep[r] = 0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) sx[k] = 0;
    auto slot_of = [&](int r) {
        int s = slot;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if ((r >> k) & 1) s ^= sx[k];
        return s;
    };
    bool have = false;
    for (int i = 0; i < n_rec; ++i) {
        if (i > 0 && i % kRecChunk == 0) {
            __syncthreads();  // the staged records are used up
            load_recs(T, recs, i, n_rec, THREADS);
            __syncthreads();
        }
        const SvRecord &rec = T.recs[i % kRecChunk];
        const int kind = __builtin_amdgcn_readfirstlane(rec.kind);
        const int a = __builtin_amdgcn_readfirstlane(rec.a), b = __builtin_amdgcn_readfirstlane(rec.b);
        if (idle && kind != SVR_GROUP) continue;
        if (kind == SVR_LAYER) {
            if (a & kSvLayerSigns) {
                uint32_t sg[R];
                sg[0] = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    sg[1 << k] = (uint32_t)__popc(base & __builtin_amdgcn_readfirstlane(rec.adj[k])) << 31;
#pragma unroll
                    for (int r = 1; r < (1 << k); ++r) sg[r | (1 << k)] = sg[r] ^ sg[1 << k];
                }
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    const uint32_t sign = sg[r] ^ ((uint32_t)(b >> r) << 31);
                    v[r] = make_double2(flip(v[r].x, sign), flip(v[r].y, sign));
                }
            }
            if (a & 1) reg_u1<K, 0>(v, rec.m[0]);
            if (a & 2) reg_u1<K, 1>(v, rec.m[1]);
            if constexpr (K > 2)
                if (a & 4) reg_u1<K, 2>(v, rec.m[2]);
        } else if (kind == SVR_GROUP) {
            if (have) {
                if (active) {
#pragma unroll
                    for (int r = 0; r < R; ++r) st[slot_of(r)] = v[r];
                }
                __syncthreads();
            }
            have = true;
            int loc = threadIdx.x;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int p = (a >> (8 * k)) & 255;
                loc = ((loc >> p) << (p + 1)) | (loc & ((1 << p) - 1));
                sx[k] = sv_slot(1 << p);
            }
            slot = sv_slot(loc);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dep[r] = 0;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if ((r >> k) & 1) dep[r] |= 1 << ((b >> (8 * k)) & 255);
            }
            gmask = dep[R - 1];
            if (active) {
                base = T.dlo[loc & 63] | T.dhi[loc >> 6] | hi;
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = st[slot_of(r)];
            }
        } else if (kind == SVR_CX) {
            if (a == 0)
                reg_cx<K, 0>(v, base, dep, gmask, b);
            else if (a == 1)
                reg_cx<K, 1>(v, base, dep, gmask, b);
            else if constexpr (K > 2)
                reg_cx<K, 2>(v, base, dep, gmask, b);
        } else if (kind == SVR_RZZ) {
            const double c = rec.m[0][0], s = ((base >> a) ^ (base >> b)) & 1 ? rec.m[0][1] : -rec.m[0][1];
#pragma unroll
            for (int r = 0; r < R; ++r)
                v[r] = cmul(v[r], make_double2(c, ((dep[r] >> a) ^ (dep[r] >> b)) & 1 ? -s : s));
        } else {  // SVR_PROJ (b: one bit)
            const int keep = __builtin_amdgcn_readfirstlane(rec.c);
            const bool drop = (b & gmask) || ((base & b) != 0) != (keep != 0);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (!(b & gmask) || ((dep[r] & b) != 0) != (keep != 0)) v[r] = drop ? make_double2(0.0, 0.0) : v[r];
        }
    }
    if (have && active) {
#pragma unroll
        for (int r = 0; r < R; ++r) st[slot_of(r)] = v[r];
    }
    __syncthreads();
}

// Index tables of a tile (local bit j -> amplitude bit lpos[j]) and, with
// prep, its product-state factors.
__device__ __forceinline__ void tile_tables(SvTables &T, const SvState &E, const SvPass &P, int tb, bool prep,
                                            int threads) {
    for (int e = threadIdx.x; e < 128; e += threads) {
        const int half = e >> 6, x = e & 63;
        const int j0 = 6 * half, j1 = min(tb, j0 + 6);
        int d = 0;
        double2 f = make_double2(1.0, 0.0), c = make_double2(0.0, 0.0);
        for (int j = j0; j < j1; ++j) {
            const int bit = (x >> (j - j0)) & 1, p = P.lpos[j];
            d |= bit << p;
            if (prep) {
                if (p < E.n) {
                    f = cmul(f, make_double2(E.init[p][2 * bit], E.init[p][2 * bit + 1]));
                    c.x += E.corr[p][2 * bit];
                    c.y += E.corr[p][2 * bit + 1];
                } else if (bit) {
                    f = make_double2(0.0, 0.0);  // padding of a small state
                }
            }
        }
        (half ? T.dhi : T.dlo)[x] = d;
        if (prep) {
            (half ? T.phi : T.plo)[x] = f;
            (half ? T.chi : T.clo)[x] = c;
        }
    }
}

// Amplitude i of the prepared tile (T.plo etc. filled) times ph (1 + c).  The
// rounding of a qubit's vector is common to all amplitudes, so unlike an
// amplitude's own rounding it does not average out of a sum over them: it is
// carried beside the factors and added once.
__device__ __forceinline__ double2 prepared(const SvTables &T, int i, double2 ph, double2 c) {
    const double2 t = cmul(cmul(T.plo[i & 63], T.phi[i >> 6]), ph);
    const double2 a = T.clo[i & 63], b = T.chi[i >> 6];
    const double x = a.x + b.x + c.x, y = a.y + b.y + c.y;
    return make_double2(t.x + (t.x * x - t.y * y), t.y + (t.x * y + t.y * x));
}

// c(s) conj(psi[s ^ m]) psi[s], real part
__device__ __forceinline__ double sv_term(double2 a, double2 b, int ny4, int sign_bits) {
    const double P = a.x * b.x + a.y * b.y, Q = a.x * b.y - a.y * b.x;
    const double v = ny4 == 0 ? P : (ny4 == 1 ? -Q : (ny4 == 2 ? -P : Q));
    return (__popc(sign_bits) & 1) ? -v : v;
}

// v's bits, lowest first, on the bits of mask, lowest first.
__device__ __forceinline__ int deposit(int64_t v, int mask) {
    int r = 0;
    while (mask && v) {
        const int low = mask & -mask;
        if (v & 1) r |= low;
        mask ^= low;
        v >>= 1;
    }
    return r;
}

// Part `part` of n_parts of instance I's outputs, by a workgroup of WAVES
// waves; psi(s) reads amplitude s.  Lane l of a wave takes the amplitudes
// whose low six bits are l, whatever these bits are: the loads are
// coalesced, lanes that differ in kept bits hold different outputs, the
// others are summed by shuffles.  A task fixes the kept bits above the low
// six; I.waves waves share the summed bits above them (each a run of the
// counted values, combined in order).
template <int WAVES, typename Psi>
__device__ __forceinline__ void measure(const SvInst &I, Psi psi, int64_t part, int64_t n_parts, double *red,
                                        double *__restrict__ outs) {
    const int k = I.n_kept, n = I.n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lanes = (1 << min(n, 6)) - 1;  // index bits the lanes spell
    const int low_rest = lanes & ~I.kept_mask;
    const int above = ((1 << n) - 1) & ~lanes;
    const int hk = above & I.kept_mask, hr = above & ~I.kept_mask;
    const int64_t n_task = int64_t(1) << __popc(hk);
    const int S = I.waves;
    const int len = (1 << __popc(hr)) / S;
    const int xm = I.xmask, zy = I.zymask, ny4 = I.n_y & 3;
    const int h0 = deposit((int64_t)(wave % S) * len, hr);
    for (int64_t t0 = part * (WAVES / S); t0 < n_task; t0 += n_parts * (WAVES / S)) {  // workgroup-uniform
        const int64_t task = t0 + wave / S;
        const bool on = task < n_task && lane <= lanes;
        const int s0 = on ? deposit(task, hk) | lane : 0;
        double acc = 0.0;
        int h = h0, t = 0;
        for (; t + 4 <= len; t += 4) {
            double2 a[4], b[4];
            int sg[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int s = s0 | h;
                b[u] = psi(s);
                a[u] = xm ? psi(s ^ xm) : b[u];
                sg[u] = s & zy;
                h = ((h | ~hr) + 1) & hr;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) acc += sv_term(a[u], b[u], ny4, sg[u]);
        }
        for (; t < len; ++t) {
            const int s = s0 | h;
            const double2 b = psi(s);
            acc += sv_term(xm ? psi(s ^ xm) : b, b, ny4, s & zy);
            h = ((h | ~hr) + 1) & hr;
        }
        if (!on) acc = 0.0;
        for (int m = 1; m <= low_rest; m <<= 1)
            if (low_rest & m) acc += __shfl_xor(acc, m, 64);
        bool put = on && (lane & low_rest) == 0;
        if (WAVES > 1 && S > 1) {
            red[threadIdx.x] = acc;
            __syncthreads();
            put = put && wave % S == 0;
            if (put)
                for (int w = 1; w < S; ++w) acc += red[threadIdx.x + 64 * w];
        }
        if (put) {
            int64_t x = 0;
            for (int j = 0; j < k; ++j) x |= (int64_t)((s0 >> I.kept_pos[j]) & 1) << (k - 1 - j);
            outs[I.out_off + x] = acc;
        }
        if (WAVES > 1 && S > 1) __syncthreads();
    }
}

// One instance per workgroup, the state in LDS throughout.
template <int K, int THREADS>
__global__ __launch_bounds__(THREADS) void k_sv_small(const SvInst *__restrict__ insts,
                                                      const SvState *__restrict__ states,
                                                      const SvPass *__restrict__ passes,
                                                      const SvRecord *__restrict__ recs, double *__restrict__ outs) {
    extern __shared__ __align__(16) double2 sv_lds[];
    __shared__ __align__(16) SvTables T;
    __shared__ double red[THREADS];
    const SvInst &I = insts[blockIdx.x];
    const SvState &E = states[I.state];
    const SvPass &P = passes[E.pass0];
    const int tb = max(E.n, K);
    load_recs(T, recs + P.rec0, 0, P.n_rec, THREADS);
    tile_tables(T, E, P, tb, true, THREADS);
    __syncthreads();
    for (int i = threadIdx.x; i < (1 << tb); i += THREADS)
        sv_lds[sv_slot(i)] = prepared(T, i, make_double2(1.0, 0.0), make_double2(0.0, 0.0));
    __syncthreads();
    run_records<K, THREADS>(sv_lds, T, recs + P.rec0, P.n_rec, tb, 0);
    auto psi = [&](int s) { return sv_lds[sv_slot(s)]; };
    measure<THREADS / 64>(I, psi, 0, 1, red, outs);
}

// Pass `pass` of the large states: workgroup (state, tile) loads its tile
// (the first pass prepares it), runs the pass's records and stores it.
template <int K, int THREADS>
__global__ __launch_bounds__(THREADS) void k_sv_pass(const SvState *__restrict__ states,
                                                     const SvPass *__restrict__ passes,
                                                     const SvRecord *__restrict__ recs, double2 *__restrict__ gstate,
                                                     int pass) {
    extern __shared__ __align__(16) double2 sv_lds[];
    __shared__ __align__(16) SvTables T;
    const SvState &E = states[blockIdx.x];
    constexpr int tb = kSvTileBits;
    const int tile = blockIdx.y;
    if (pass >= E.n_pass || tile >= (1 << (E.n - tb))) return;  // whole workgroup: before any barrier
    const SvPass &P = passes[E.pass0 + pass];
    load_recs(T, recs + P.rec0, 0, P.n_rec, THREADS);
    tile_tables(T, E, P, tb, pass == 0, THREADS);
    int hi = 0;
    double2 ph = make_double2(1.0, 0.0), pc = make_double2(0.0, 0.0);
    for (int j = 0; j < E.n - tb; ++j) {
        const int bit = (tile >> j) & 1, p = P.hpos[j];
        hi |= bit << p;
        if (pass == 0) {
            ph = cmul(ph, make_double2(E.init[p][2 * bit], E.init[p][2 * bit + 1]));
            pc.x += E.corr[p][2 * bit];
            pc.y += E.corr[p][2 * bit + 1];
        }
    }
    __syncthreads();
    double2 *g = gstate + E.off;
    if (pass == 0) {
        for (int i = threadIdx.x; i < (1 << tb); i += THREADS)
            sv_lds[sv_slot(i)] = prepared(T, i, ph, pc);
    } else {
#pragma unroll 4
        for (int i = threadIdx.x; i < (1 << tb); i += THREADS)
            sv_lds[sv_slot(i)] = g[T.dlo[i & 63] | T.dhi[i >> 6] | hi];
    }
    __syncthreads();
    run_records<K, THREADS>(sv_lds, T, recs + P.rec0, P.n_rec, tb, hi);
#pragma unroll 4
    for (int i = threadIdx.x; i < (1 << tb); i += THREADS)
        g[T.dlo[i & 63] | T.dhi[i >> 6] | hi] = sv_lds[sv_slot(i)];
}

// Outputs of the large instances: workgroup (instance, part).
constexpr int kMeasThreads = 64 * kSvMeasWaves;
__global__ __launch_bounds__(kMeasThreads) void k_sv_measure(const SvInst *__restrict__ insts,
                                                             const SvState *__restrict__ states,
                                                             const double2 *__restrict__ gstate,
                                                             double *__restrict__ outs) {
    __shared__ double red[kMeasThreads];
    const SvInst &I = insts[blockIdx.x];
    const double2 *__restrict__ g = gstate + states[I.state].off;
    auto psi = [&](int s) { return g[s]; };
    measure<kSvMeasWaves>(I, psi, blockIdx.y, gridDim.y, red, outs);
}

// entries[e] = sum over e's terms t (in order) of coef[t] * outs[term_out[t]]
__global__ __launch_bounds__(256) void k_qt_assemble(const int64_t *__restrict__ start,
                                                     const int64_t *__restrict__ term_out,
                                                     const double *__restrict__ coef, int64_t n_entries,
                                                     const double *__restrict__ outs, double *__restrict__ entries) {
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n_entries; e += (int64_t)gridDim.x * 256) {
        double acc = 0.0;
        for (int64_t t = start[e]; t < start[e + 1]; ++t) acc += coef[t] * outs[term_out[t]];
        entries[e] = acc;
    }
}

}  // namespace

template <int K, int THREADS>
static hipError_t go_small(const SvLaunch &L, const SvClass &c, double *outs, hipStream_t st) {
    const int lds = (int)sizeof(double2) << std::max(c.max_n, K);
    const hipError_t e =
        hipFuncSetAttribute((const void *)k_sv_small<K, THREADS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e;
    }
    hipLaunchKernelGGL((k_sv_small<K, THREADS>), dim3((unsigned)c.n_insts), dim3(THREADS), lds, st,
                       L.insts + c.inst0, L.states, L.passes, L.recs, outs);
    return hipGetLastError();
}

hipError_t launch_sv_eval(const SvLaunch &L, double *outs, hipStream_t st) {
    hipError_t e = hipSuccess;
    if (L.cls[0].n_insts > 0) e = go_small<kSvRegBits0, kSvThreads0>(L, L.cls[0], outs, st);
    if (e == hipSuccess && L.cls[1].n_insts > 0) e = go_small<kSvRegBits1, kSvThreads1>(L, L.cls[1], outs, st);
    if (e != hipSuccess || L.cls[2].n_insts <= 0) return e;
    const SvClass &c = L.cls[2];
    constexpr int lds = (int)sizeof(double2) << kSvTileBits;
    e = hipFuncSetAttribute((const void *)k_sv_pass<kSvRegBits2, kSvThreads2>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e;
    }
    const unsigned tiles = 1u << (c.max_n - kSvTileBits);
    for (int p = 0; p < L.n_pass; ++p)
        hipLaunchKernelGGL((k_sv_pass<kSvRegBits2, kSvThreads2>), dim3((unsigned)L.n_large, tiles),
                           dim3(kSvThreads2), lds, st, L.states + L.large0, L.passes, L.recs, L.gstate, p);
    hipLaunchKernelGGL(k_sv_measure, dim3((unsigned)c.n_insts, (unsigned)c.parts), dim3(kMeasThreads), 0, st,
                       L.insts + c.inst0, L.states, L.gstate, outs);
    return hipGetLastError();
}

hipError_t launch_qt_assemble(const int64_t *start, const int64_t *term_out, const double *coef, int64_t n_entries,
                              const double *outs, double *entries, hipStream_t st) {
    if (n_entries <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n_entries + 255) / 256, 4096);
    hipLaunchKernelGGL(k_qt_assemble, dim3((unsigned)blocks), dim3(256), 0, st, start, term_out, coef, n_entries,
                       outs, entries);
    return hipGetLastError();
}

}  // namespace kern
}  // namespace htn
