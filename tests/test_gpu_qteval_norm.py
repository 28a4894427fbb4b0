"""Norms of evaluated states.

Unitaries merged on the host are rounded once for all amplitudes, so that their
error of the norm (some 1e-16 each, twice that in a probability) adds up over a
state's unitaries instead of averaging out over its amplitudes: 4.6e-16 to
5.5e-16, root mean square of the states below.  An evaluator that applies every
unitary by itself is at 1.5e-16 to 2.4e-16 (6 to 13 qubits, 96 and 24 states a
size); the bound lies 25 % above, two standard errors of 24 states."""

import math

import numpy as np
import pytest

from paper_2410_15080_amd import qteval
from workloads import circuits as c

pytestmark = pytest.mark.gpu


def _instance(rng, n):
    """Two unitaries on every qubit (merged by the evaluator) between layers of
    CZ gates, all qubits kept."""
    ops = []
    for layer in range(3):
        for q in range(n):
            ops += [("u", q, c.ry(rng.uniform(0, 2 * np.pi))), ("u", q, c.rz(rng.uniform(0, 2 * np.pi)))]
        ops += [("cz", q, q + 1) for q in range(layer % 2, n - 1, 2)]
    return c.Instance(n, [np.array([1.0, 0.0]) if q % 2 else np.array([0.6, 0.8]) for q in range(n)], ops, "I" * n,
                      list(range(n)))


def _norm(inst):
    """Squared norm in 80 bits (the gates are unitary to FP64 only)."""
    n = inst.n_qubits
    psi = np.array(1, dtype=np.clongdouble)
    for v in inst.init:
        psi = np.multiply.outer(psi, v.astype(np.clongdouble))
    for op in inst.ops:
        if op[0] == "u":
            u = np.asarray(op[2]).astype(np.clongdouble)
            a, b = np.take(psi, 0, op[1]), np.take(psi, 1, op[1])
            psi = np.stack([u[0, 0] * a + u[0, 1] * b, u[1, 0] * a + u[1, 1] * b], axis=op[1])
        else:
            ix = [slice(None)] * n
            ix[op[1]] = ix[op[2]] = 1
            psi = psi.copy()
            psi[tuple(ix)] *= -1
    return (psi.real ** 2 + psi.imag ** 2).sum()


# one wave, one workgroup, tiles in device memory
@pytest.mark.parametrize("n", [8, 12, 13])
def test_norm_of_merged_unitaries(n):
    import torch
    rng = np.random.default_rng(n)
    insts = [_instance(rng, n) for _ in range(24)]
    (got,) = qteval.Evaluator([c.QTSpec((len(insts) << n,), insts,
                                        [[(k, x, 1.0)] for k in range(len(insts)) for x in range(1 << n)])]).run()
    torch.cuda.synchronize()
    out = got.cpu().numpy().reshape(len(insts), -1)
    err = [float(np.longdouble(math.fsum(o)) / _norm(i) - 1) for o, i in zip(out, insts)]
    rms = float(np.sqrt(np.mean(np.square(err))))
    assert rms <= 3e-16, (rms, err)
