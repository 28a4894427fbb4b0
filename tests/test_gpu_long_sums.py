"""Rounding error of long sums in the fused kernel's matrix-core steps.

The terms are positive, so n additions to a running sum S of equal steps leave
an error of 0.41 u S sqrt(n / 3) (root mean square; u = 2^-53 or 2^-24, 0.41 u
that of one rounding).  With 32 terms joined before they are added, a sum of K
terms takes n = K / 32 such additions, the sums of the 32 terms themselves and of
the workgroup's K ranges adding little to it; a chain of all K terms in two
accumulators takes four times that error and more."""

import json

import numpy as np
import pytest

from paper_2410_15080_amd import htn
from workloads.network import Network

from gpu_helpers import contract, create

pytestmark = pytest.mark.gpu


# several blocks a wave, one block a wave, K split over the workgroup's waves
@pytest.mark.parametrize("threads,M,N,K,ranges", [(64, 64, 64, 8192, 1), (256, 48, 48, 8192, 1), (512, 16, 16, 49152, 8)])
@pytest.mark.parametrize("compute", [htn.HTN_F64, htn.HTN_F32])
def test_error_of_a_long_sum(compute, threads, M, N, K, ranges):
    rng = np.random.default_rng(K + M)
    dt, u = (np.float64, 2.0 ** -53) if compute == htn.HTN_F64 else (np.float32, 2.0 ** -24)
    a, b = (rng.uniform(1, 2, size=s).astype(dt) for s in ((M, K), (K, N)))
    w = Network([a.astype(np.float64), b.astype(np.float64)], [[0, 2], [2, 1]], [M, N, K], [0, 1])
    net = create(w, compute=compute, storage=htn.HTN_F64, exec_mode=htn.HTN_EXEC_FUSED)
    htn.htn_set_option(net, htn.HTN_OPT_FUSED_THREADS, threads)
    step = json.loads(htn.htn_plan_json(net))["steps"][-1]
    assert step["tile"] and step["tcfg"][0] == 0
    ref = a.astype(np.longdouble) @ b.astype(np.longdouble)
    err = (contract(net, (M, N)) - ref) / ref
    rms = float(np.sqrt((err.astype(np.float64) ** 2).mean()))
    assert rms <= u * (0.5 * np.sqrt(K / ranges / 32 / 3) / np.sqrt(ranges) + 1.0), rms / u
