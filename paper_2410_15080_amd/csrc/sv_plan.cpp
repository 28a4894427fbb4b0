// Scheduling of statevector ops into register groups and tile passes (see
// sv_plan.hpp).
#include "sv_plan.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace htn {

namespace {

// Ops looked ahead (in program order) when a group or a tile is chosen: the
// search stays linear in the number of ops.
constexpr int kWindow = 256;

enum { U1, CZ, CX, RZZ, PROJ };

struct Op {
    int kind;
    int need = -1;  // amplitude bit that must be a register bit (-1: none)
    int p0 = 0, p1 = 0;
    double m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int bit = 0;  // PROJ: the value kept
};

// An op not yet run, as masks of amplitude bits: those that it changes, those
// that it is diagonal in (or controlled by), those that must be register bits,
// and those of which one must be (0: none).  Its order is kept against every
// earlier op that changes one of its bits, or that touches the one it changes.
struct Left {
    uint32_t chg = 0, dia = 0, req = 0, any = 0;
    int op = 0;
};

// c = a * b, 2x2 complex row-major (re, im)
void mul2(const double *a, const long double *b, long double *c) {
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            long double re = 0.0L, im = 0.0L;
            for (int k = 0; k < 2; ++k) {
                const double *x = a + 4 * i + 2 * k;
                const long double *y = b + 4 * k + 2 * j;
                re += x[0] * y[0] - x[1] * y[1];
                im += x[0] * y[1] + x[1] * y[0];
            }
            c[4 * i + 2 * j] = re;
            c[4 * i + 2 * j + 1] = im;
        }
}

// Re tr(M^* (M - m)) / tr(M^* M): what rounding M to m takes from the norm of a
// state on whose qubit nothing else is known.
long double norm_lost(const long double *M, const double *m) {
    long double d = 0.0L, s = 0.0L;
    for (int i = 0; i < 8; ++i) {
        d += M[i] * (M[i] - m[i]);
        s += M[i] * M[i];
    }
    return std::abs(d) < 1e-15L * s ? d / s : 0.0L;  // (no for zeros, infinities and NaN)
}

struct Scheduler {
    std::vector<Op> ops;
    std::vector<Left> left;  // program order
    uint32_t bits = 0;       // bits that any op acts on

    // Worth of the ops that can run with register (or tile) bits `set`, in
    // program order within the window; `order`, if given, receives their
    // places in `left`.  A CZ waits for one of its bits.  An op that cannot
    // run holds up the later ones that do not commute with it.
    int trial(uint32_t set, std::vector<int> *order) const {
        const int end = std::min((int)left.size(), kWindow);
        uint32_t held = 0, held_chg = 0;  // bits of ops held up; those that they change
        int n = 0;
        for (int i = 0; i < end; ++i) {
            const Left &o = left[i];
            if ((o.req & ~set) || (o.any && !(o.any & set)) || (o.chg & held) || (o.dia & held_chg)) {
                held |= o.chg | o.dia;
                held_chg |= o.chg;
                if (held_chg == bits) break;  // nothing commutes with all that is held up
                continue;
            }
            n += o.req ? 4 : 1;
            if (order) order->push_back(i);
        }
        return n;
    }
    // `count` bits out of `from`, starting from `set`: each time the bit
    // that lets the most ops run (the lowest among equals).
    uint32_t choose(uint32_t from, uint32_t set, int count) {
        while (__builtin_popcount(set) < count) {
            int best = -1, best_n = -1;
            for (int p = 0; p < 32; ++p) {
                if (!((from >> p) & 1) || ((set >> p) & 1)) continue;
                const int n = trial(set | (1u << p), nullptr);
                if (n > best_n) {
                    best_n = n;
                    best = p;
                }
            }
            set |= 1u << best;
        }
        return set;
    }
    // the ops at these places of `left` have run
    void finish(const std::vector<int> &run) {
        size_t r = 0, w = 0;
        for (size_t i = 0; i < left.size(); ++i) {
            if (r < run.size() && run[r] == (int)i)
                ++r;
            else
                left[w++] = left[i];
        }
        left.resize(w);
    }
};

// The records of one group's ops (program order; reg[p]: register bit of
// amplitude bit p, or -1).
void emit_group(const Scheduler &S, const std::vector<int> &run, const std::vector<int> &reg, int K,
                std::vector<SvRecord> &recs) {
    std::vector<SvRecord> layers;
    int u_next[kSvMaxRegBits], z_next[kSvMaxRegBits];  // first layer a unitary / a CZ on the bit may join
    auto fresh = [] {
        SvRecord x;
        std::memset(&x, 0, sizeof(x));
        x.kind = SVR_LAYER;
        return x;
    };
    auto layer = [&](int l) -> SvRecord & {
        while ((int)layers.size() <= l) layers.push_back(fresh());
        return layers[l];
    };
    auto close = [&] {
        recs.insert(recs.end(), layers.begin(), layers.end());
        layers.clear();
        for (int k = 0; k < kSvMaxRegBits; ++k) u_next[k] = z_next[k] = 0;
    };
    close();
    for (int i : run) {
        const Op &o = S.ops[S.left[i].op];
        if (o.kind == U1) {
            const int k = reg[o.p0], l = u_next[k];
            SvRecord &x = layer(l);
            x.a |= 1 << k;
            std::memcpy(x.m[k], o.m, sizeof(o.m));
            u_next[k] = z_next[k] = l + 1;
        } else if (o.kind == CZ) {
            const int k0 = reg[o.p0], k1 = reg[o.p1];
            const int l = std::max(k0 >= 0 ? z_next[k0] : 0, k1 >= 0 ? z_next[k1] : 0);
            SvRecord &x = layer(l);
            x.a |= kSvLayerSigns;
            if (k0 >= 0 && k1 >= 0) {
                for (int r = 0; r < (1 << K); ++r)
                    if (((r >> k0) & 1) && ((r >> k1) & 1)) x.b ^= 1 << r;
            } else {
                x.adj[k0 >= 0 ? k0 : k1] ^= 1 << (k0 >= 0 ? o.p1 : o.p0);
            }
            // the signs come before the layer's unitaries
            for (int k : {k0, k1})
                if (k >= 0) u_next[k] = std::max(u_next[k], l);
        } else {
            close();
            SvRecord x = fresh();
            std::memcpy(x.m[0], o.m, sizeof(o.m));
            if (o.kind == CX) {
                x.kind = SVR_CX;
                x.a = reg[o.p1];
                x.b = 1 << o.p0;
            } else if (o.kind == RZZ) {
                x.kind = SVR_RZZ;
                x.a = o.p0;
                x.b = o.p1;
            } else {
                x.kind = SVR_PROJ;
                x.b = 1 << o.p0;
                x.c = o.bit;
            }
            recs.push_back(x);
        }
    }
    close();
}

}  // namespace

SvSchedule sv_schedule(int n, const htn_sv_op *in, int n_ops, int tile, int K) {
    SvSchedule out;
    const int nb = std::max(n, K);  // amplitude bits (bits n.. of a padded small state stay 0)
    static const long double one[8] = {1, 0, 0, 0, 0, 0, 1, 0};
    out.lead.resize(8 * (size_t)n);
    for (int q = 0; q < n; ++q) std::copy(one, one + 8, &out.lead[8 * (size_t)q]);
    Scheduler S;
    // consecutive single-qubit unitaries of a qubit become one matrix
    std::vector<long double> pend(8 * (size_t)n);
    std::vector<char> has(n, 0), touched(n, 0);
    auto push = [&](Op o) { S.ops.push_back(std::move(o)); };
    auto flush = [&](int q) {
        if (has[q]) {
            if (!touched[q]) {
                std::copy_n(&pend[8 * (size_t)q], 8, &out.lead[8 * (size_t)q]);
            } else {
                Op o;
                o.kind = U1;
                o.need = o.p0 = n - 1 - q;
                std::copy_n(&pend[8 * (size_t)q], 8, o.m);
                out.lost += norm_lost(&pend[8 * (size_t)q], o.m);
                push(o);
            }
            has[q] = 0;
        }
        touched[q] = 1;
    };
    for (int k = 0; k < n_ops; ++k) {
        const htn_sv_op &x = in[k];
        if (x.kind == HTN_SV_U1) {
            long double *p = &pend[8 * (size_t)x.q0];
            if (has[x.q0]) {
                long double t[8];
                mul2(x.m, p, t);
                std::copy_n(t, 8, p);
            } else {
                std::copy_n(x.m, 8, p);
            }
            has[x.q0] = 1;
            continue;
        }
        flush(x.q0);
        Op o;
        o.p0 = n - 1 - x.q0;
        if (x.kind == HTN_SV_PROJ) {
            o.kind = PROJ;
            o.bit = x.q1;
        } else {
            flush(x.q1);
            o.p1 = n - 1 - x.q1;
            o.kind = x.kind == HTN_SV_CZ ? CZ : (x.kind == HTN_SV_CX ? CX : RZZ);
            if (x.kind == HTN_SV_CX) o.need = o.p1;  // the control may be any bit
            if (x.kind == HTN_SV_RZZ) {
                o.m[0] = std::cos(0.5 * x.m[0]);
                o.m[1] = std::sin(0.5 * x.m[0]);
            }
        }
        push(o);
    }
    for (int q = 0; q < n; ++q) flush(q);
    for (int i = 0; i < (int)S.ops.size(); ++i) {
        const Op &o = S.ops[i];
        Left l;
        l.op = i;
        if (o.need >= 0) l.req = l.chg = 1u << o.need;
        if (o.kind != U1) l.dia |= 1u << o.p0;
        if (o.kind == CZ || o.kind == RZZ) l.dia |= 1u << o.p1;
        if (o.kind == CZ) l.any = l.dia;
        S.bits |= l.chg | l.dia;
        S.left.push_back(l);
    }
    const uint32_t all = nb >= 32 ? ~0u : (1u << nb) - 1;
    // a tile holds the three lowest bits: 128-byte runs of the state
    const uint32_t low = std::min<uint32_t>(all, 7u);
    do {
        const uint32_t tset = tile >= nb ? all : S.choose(all, low, tile);
        SvSchedule::Pass P;
        std::vector<int> local(32, -1);
        for (int p = 0; p < nb; ++p) {
            if ((tset >> p) & 1) {
                local[p] = (int)P.lpos.size();
                P.lpos.push_back(p);
            } else {
                P.hpos.push_back(p);
            }
        }
        while (!S.left.empty()) {
            const uint32_t rset = S.choose(tset, 0, K);
            std::vector<int> run;
            S.trial(rset, &run);
            if (run.empty()) break;  // the rest needs another tile
            SvRecord g;
            std::memset(&g, 0, sizeof(g));
            g.kind = SVR_GROUP;
            std::vector<int> reg(32, -1);
            int r = 0;
            for (int p = 0; p < nb; ++p)
                if ((rset >> p) & 1) {
                    g.a |= local[p] << (8 * r);
                    g.b |= p << (8 * r);
                    reg[p] = r++;
                }
            P.recs.push_back(g);
            emit_group(S, run, reg, K, P.recs);
            S.finish(run);
        }
        out.passes.push_back(std::move(P));
    } while (!S.left.empty());
    return out;
}

}  // namespace htn
