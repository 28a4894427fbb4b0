"""Tiled steps on the matrix cores outside the fused kernel: one launch per
step, the work queue's and the level launches' items.

The inputs are multiples of 1/64 up to 1 (exact in BF16), so every product is
a multiple of 2^-12 and every sum of up to 4096 of them is exact in FP32: the
results must be equal, whatever the order of the additions."""

import json

import numpy as np
import pytest

from paper_2410_15080_amd import htn
from workloads.network import Network

from gpu_helpers import create
from test_gpu_queue import _run_batch

pytestmark = pytest.mark.gpu

# (M, N, K): the smallest sides, one past and one short of a block and of each
# tile shape, K around its chunks (16, 32) and split into ranges with a short
# last one
SHAPES = [(4, 256, 8), (256, 5, 9), (16, 64, 15), (64, 17, 16), (65, 31, 17), (33, 48, 31), (32, 97, 32), (15, 80, 33),
          (130, 6, 63), (31, 33, 64), (96, 64, 129), (36, 24, 1000), (64, 16, 4096), (576, 36, 3456)]


def _net(rng, M, N, K, flip):
    a, b = (rng.integers(-64, 65, size=s) / 64.0 for s in ((M, K), (K, N)))
    return Network([a, b], [[0, 2], [2, 1]], [M, N, K], [1, 0] if flip else [0, 1]), (a @ b).T if flip else a @ b


@pytest.mark.parametrize("compute", [htn.HTN_F64, htn.HTN_F32, htn.HTN_BF16])
def test_tiled_steps_are_exact(compute):
    rng = np.random.default_rng(5)
    ws, refs = zip(*[_net(rng, *s, flip) for s in SHAPES for flip in (False, True)])
    for mode in (0, 1, 2):  # levels (or the queue for small steps), queue, a launch per step
        nets = [create(w, compute=compute, final_sum=htn.HTN_SUM_PLAIN, storage=htn.HTN_F64,
                       exec_mode=htn.HTN_EXEC_STEPS) for w in ws]
        for n in nets:
            htn.htn_set_option(n, htn.HTN_OPT_FUSED_THREADS, 64)
            htn.htn_set_option(n, htn.HTN_OPT_QUEUE, mode)
        plans = [json.loads(htn.htn_plan_json(n))["steps"][-1] for n in nets]
        assert all(p["xtile"][0] or p["mfma"] for p in plans)
        assert {p["xtile"][2] for p in plans} == {0, 1, 2} and {p["xtile"][3] for p in plans} == {0, 1}
        assert any(p["xtile"][1] > 1 for p in plans)
        outs = [htn.new_output(n) for n in nets]
        b, r = _run_batch(nets, outs)
        htn.htn_batch_destroy(b)
        for i, (got, ref) in enumerate(zip(r[0], refs)):
            assert np.array_equal(got.astype(np.float64).reshape(ref.shape), ref), (mode, i, SHAPES[i // 2])


@pytest.mark.parametrize("compute", [htn.HTN_F32, htn.HTN_BF16])
def test_products_into_fp64_are_exact(compute):
    """Packed products with an FP64 result: sums of one chunk (up to 64 terms)
    and of more, rows of whole 128-byte lines and ragged ones."""
    rng = np.random.default_rng(6)
    for M, N, K in [(800, 672, 8), (301, 272, 63), (257, 259, 64), (272, 256, 65), (300, 129, 130)]:
        w, ref = _net(rng, M, N, K, False)
        n = create(w, compute=compute, final_sum=htn.HTN_SUM_FP64, storage=htn.HTN_F64, exec_mode=htn.HTN_EXEC_STEPS)
        p = json.loads(htn.htn_plan_json(n))["steps"][-1]
        assert p["mfma"] and not p["xtile"][0]
        import torch
        out = htn.new_output(n)
        htn.htn_contract(n, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().reshape(M, N), ref), (M, N, K)


@pytest.mark.parametrize("compute", [htn.HTN_F64, htn.HTN_F32, htn.HTN_BF16])
def test_final_product_in_either_output_order(compute):
    """A large final product is a matrix product whichever of its operands the
    output's labels begin with; the fused kernel, asked for, still takes both."""
    import torch
    rng = np.random.default_rng(8)
    for flip in (False, True):
        w, ref = _net(rng, 300, 420, 48, flip)
        n = create(w, compute=compute, final_sum=htn.HTN_SUM_FP64, storage=htn.HTN_F64)
        assert json.loads(htn.htn_plan_json(n))["steps"][-1]["mfma"]
        for mode in (htn.HTN_EXEC_STEPS, htn.HTN_EXEC_FUSED, htn.HTN_EXEC_AUTO):
            htn.htn_set_option(n, htn.HTN_OPT_EXEC, mode)
            out = htn.new_output(n)
            htn.htn_contract(n, out)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().reshape(ref.shape), ref), (flip, mode)
