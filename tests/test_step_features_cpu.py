"""Step features name the kernel that runs the step (no GPU)."""

import json

import numpy as np
import pytest

from paper_2410_15080_amd import htn


def _lg(v):
    return np.float32(np.log2(max(v, 1.0)) / 8.0)


@pytest.mark.parametrize("M,N,K", [(96, 64, 129), (36, 24, 1000), (256, 5, 9), (64, 16, 4096)])
def test_tiled_step_outside_the_fused_kernel(M, N, K):
    net = htn.htn_create([np.zeros((M, K)), np.zeros((K, N))], [[0, 2], [2, 1]], [M, N, K], [0, 1])
    fused = htn.htn_step_features(net)[-1]
    htn.htn_set_option(net, htn.HTN_OPT_EXEC, htn.HTN_EXEC_STEPS)
    x = htn.htn_step_features(net)[-1]
    step = json.loads(htn.htn_plan_json(net))["steps"][-1]
    assert step["xtile"][0] and not step["mfma"]
    assert fused[21] == 1 and x[21] == 0
    assert list(x[5:10]) == [_lg(M), _lg(N), _lg(K), _lg(16), _lg(step["xtile"][1])]
    # a tiled matrix-core step, and neither one nor several lanes per output
    assert list(x[10:15]) == [1, 0, 0, 0, 1]
