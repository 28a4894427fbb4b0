"""The per-step workspace stays within the allocation-free entry point's where
only the K ranges of a tiled step would take it beyond (no GPU)."""

import json

import numpy as np
import pytest

from paper_2410_15080_amd import htn

SCRATCH = 64 * 1024 * 1024


# an outer product of d x d values, held while a 60 x 60 product of 4096 terms
# (64 ranges of 28 800 bytes) runs: below the limit with the ranges, below it
# without them only, and above it either way
@pytest.mark.parametrize("d,fits,split", [(2700, True, True), (2850, True, False), (2890, False, True)])
def test_ranges_do_not_cost_the_allocation_free_workspace(d, fits, split):
    M, K = 60, 4096
    net = htn.htn_create([np.zeros(s) for s in ((d, 2), (2, d), (M, K), (K, M), (d,), (d,))],
                         [[0, 1], [1, 2], [3, 4], [4, 5], [0], [2]], [d, 2, d, M, K, M], [3, 5])
    htn.htn_set_path(net, [(0, 1), (2, 3), (6, 4), (8, 5), (9, 7)])
    step = json.loads(htn.htn_plan_json(net))["steps"][1]
    assert step["xtile"][0] and (step["xtile"][1] > 1) == split
    assert (htn.htn_get_info(net).workspace_bytes <= SCRATCH) == fits
