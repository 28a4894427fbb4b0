// Schedule of a statevector instance's ops for the QT evaluator's kernels
// (qteval.hip).  Host-only C++.
//
// The kernels hold 2^K amplitudes of a state per thread: a group fixes K
// amplitude-index bits as register bits, and every op whose changed bit is
// one of them (diagonal ops and controls: any bits) runs on registers
// before the amplitudes go back to LDS.  Inside a group the CZ gates and
// the single-qubit unitaries are packed into layers (all CZs of a layer are
// one sign per amplitude, then at most one unitary per register bit): a
// record costs its branches as much as its arithmetic, so few and large
// ones.  A state of more qubits than a tile has bits is worked through in
// passes over tiles.
#pragma once

#include <cstdint>
#include <vector>

#include "htn.h"

namespace htn {

// GROUP: a, b: the register bits' positions in the tile and in the amplitude
//   index, one byte each, ascending.
// LAYER: a: bit k set: unitary m[k] on register bit k, after the signs; with
//   bit 8 set, signs: the amplitude of register r is negated if the parity
//   of (index & adj[k]) summed over the bits k of r, plus bit r of b, is odd.
// CX: a: register bit of the target, b: mask of the control.
// RZZ: a, b: amplitude bits, m[0][0..1]: cos and sin of the half angle.
// PROJ: b: mask of the bit, c: the value kept.
enum { SVR_GROUP = 0, SVR_LAYER = 1, SVR_CX = 2, SVR_RZZ = 3, SVR_PROJ = 4 };
constexpr int kSvMaxRegBits = 3;
constexpr int kSvLayerSigns = 256;

struct SvRecord {
    int32_t kind;
    int32_t a, b, c;
    int32_t adj[4];
    double m[kSvMaxRegBits][8];
};
static_assert(sizeof(SvRecord) == 224, "copied to the device as 16-byte chunks");

struct SvSchedule {
    // per qubit, the product of the single-qubit unitaries ahead of every
    // other op on it (row-major, re/im): applied to its initial vector
    std::vector<long double> lead;
    // relative loss of norm by rounding the other merged unitaries, in all
    long double lost = 0.0L;
    struct Pass {
        std::vector<int> lpos, hpos;  // amplitude bits of the tile, and of the tile number (ascending)
        std::vector<SvRecord> recs;
    };
    std::vector<Pass> passes;  // at least one
};

// Schedule of the n_ops ops of an n-qubit instance (validated by the caller), n
// at least 1.  K: register bits of a group, 1 to kSvMaxRegBits; a state of
// fewer qubits is padded to K bits, which stay 0.  tile: amplitude bits that a
// workgroup holds, at least max(3, K), since the three lowest bits are in every
// tile; max(n, K) or more gives one pass over the whole state.
SvSchedule sv_schedule(int n, const htn_sv_op *ops, int n_ops, int tile, int K);

}  // namespace htn
