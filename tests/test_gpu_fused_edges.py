"""Fused steps at the edges of their tiles: one product A[k, m] B[k, n] per
network (two tensors, optionally a third that makes it an intermediate),
against numpy.

Tolerance: |x_hat - x| <= 2 (K + 2) u sum_k |a b| for a product of K terms in
any order (u = 2^-53 FP64, 2^-24 FP32), twice over for the second product."""

import numpy as np
import pytest

from paper_2410_15080_amd import htn

pytestmark = pytest.mark.gpu

U = {"float64": 2.0 ** -53, "float32": 2.0 ** -24}


def _run(tensors, labels, dims, out, dtype, threads, lds):
    import torch
    code = htn.HTN_F64 if dtype == "float64" else htn.HTN_F32
    ts = [torch.from_numpy(t.astype(dtype)).cuda() for t in tensors]
    net = htn.htn_create(ts, labels, dims, out, compute=code)
    htn.htn_set_option(net, htn.HTN_OPT_EXEC, htn.HTN_EXEC_FUSED)
    htn.htn_set_option(net, htn.HTN_OPT_FUSED_THREADS, threads)
    htn.htn_set_option(net, htn.HTN_OPT_FUSED_LDS_BYTES, lds)
    res = htn.new_output(net)
    htn.htn_contract(net, res)
    torch.cuda.synchronize()
    return res.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("threads,lds", [(64, 65536), (256, 65536), (512, 163840), (256, 20480)])
def test_product_edges(dtype, threads, lds):
    """M, N at the edges of 16 and 32 blocks, K at those of slices of 4, pairs
    and stages of 16; the smallest budget keeps operands outside LDS."""
    rng = np.random.default_rng(threads + lds)
    for m, n, k in [(16, 16, 4), (16, 17, 5), (17, 16, 7), (31, 33, 8), (33, 31, 12), (64, 48, 15), (48, 64, 16),
                    (65, 63, 20), (80, 96, 23), (96, 80, 33), (128, 112, 40), (4, 64, 6), (300, 5, 9), (1, 640, 3)]:
        a = rng.uniform(-1, 1, (k, m)).astype(dtype).astype(np.float64)
        b = rng.uniform(-1, 1, (k, n)).astype(dtype).astype(np.float64)
        got = _run([a, b], [[0, 1], [0, 2]], [k, m, n], [2, 1], dtype, threads, lds).reshape(n, m)
        bound = 2 * (k + 2) * U[dtype] * (np.abs(b).T @ np.abs(a))
        assert (np.abs(got - b.T @ a) <= bound).all(), (m, n, k)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_intermediate_digits(dtype):
    """An intermediate whose consumer interleaves the labels of M and N (several
    digits a side, extents 1 to 7), then summed away by a third tensor."""
    rng = np.random.default_rng(5)
    dims = [7, 3, 4, 6, 1, 5, 4, 2]  # 0: summed first; 1, 3, 4, 6 from A; 2, 5, 7 from B
    a = rng.uniform(-1, 1, [dims[l] for l in (1, 0, 3, 4, 6)]).astype(dtype).astype(np.float64)
    b = rng.uniform(-1, 1, [dims[l] for l in (2, 5, 0, 7)]).astype(dtype).astype(np.float64)
    c = rng.uniform(-1, 1, [dims[l] for l in (5, 1, 6, 2)]).astype(dtype).astype(np.float64)
    labels = [[1, 0, 3, 4, 6], [2, 5, 0, 7], [5, 1, 6, 2]]
    got = _run([a, b, c], labels, dims, [7, 3, 4], dtype, 256, 65536)
    ref = np.einsum(a, labels[0], b, labels[1], c, labels[2], [7, 3, 4])
    mag = np.einsum(np.abs(a), labels[0], np.abs(b), labels[1], np.abs(c), labels[2], [7, 3, 4])
    n_terms = dims[0] + dims[1] * dims[2] * dims[5] * dims[6]
    assert (np.abs(got - ref.ravel()) <= 2 * (n_terms + 4) * U[dtype] * mag.ravel()).all()


@pytest.mark.parametrize("final", [htn.HTN_SUM_PLAIN, htn.HTN_SUM_COMPENSATED])
@pytest.mark.parametrize("dims", [(1, 1), (1, 63), (8, 8), (7, 73), (9, 57), (17, 241), (144, 144)])
def test_long_sums(final, dims):
    """One output by a whole workgroup and by a wave: sums around the number of
    terms read ahead (two labels: one table of 4097 entries would not fit the
    smallest LDS budget)."""
    import torch
    n_sum = dims[0] * dims[1]
    rng = np.random.default_rng(n_sum)
    a, b = rng.uniform(-1, 1, n_sum), rng.uniform(-1, 1, n_sum)
    for threads, lds in ((64, 65536), (512, 163840), (256, 20480)):
        net = htn.htn_create([torch.from_numpy(x.reshape(dims)).cuda() for x in (a, b)], [[0, 1], [0, 1]], list(dims),
                             [], final_sum=final)
        htn.htn_set_option(net, htn.HTN_OPT_EXEC, htn.HTN_EXEC_FUSED)
        htn.htn_set_option(net, htn.HTN_OPT_FUSED_THREADS, threads)
        htn.htn_set_option(net, htn.HTN_OPT_FUSED_LDS_BYTES, lds)
        out = htn.new_output(net)
        htn.htn_contract(net, out)
        torch.cuda.synchronize()
        import math
        ref = math.fsum(x * y for x, y in zip(a, b))
        assert abs(float(out.item()) - ref) <= 2 * (n_sum + 2) * 2.0 ** -53 * np.abs(a * b).sum()


def test_index_outside_lds():
    """A budget that takes the program without its index: the index is read from
    device memory, the values live outside LDS; same sums, same result."""
    import json
    import torch
    from workloads import configs
    w = configs.grid_network(3)
    vals = []
    ts = [torch.from_numpy(np.asarray(t, dtype=np.float64)).cuda() for t in w.tensors]
    for tight in (False, True):
        net = htn.htn_create(ts, w.labels, w.dims, w.out_labels)
        htn.htn_set_option(net, htn.HTN_OPT_EXEC, htn.HTN_EXEC_FUSED)
        if tight:
            prog = json.loads(htn.htn_plan_json(net))["program"]
            words = prog[0] - (1 + 6 * prog[prog[2]])  # 256 threads: six index words a phase
            htn.htn_set_option(net, htn.HTN_OPT_FUSED_LDS_BYTES, ((words + 3) // 4 * 4 + 2 * prog[4]) * 4 + 256)
            prog = json.loads(htn.htn_plan_json(net))["program"]
            assert prog[2] >= prog[0]
        out = htn.new_output(net)
        htn.htn_contract(net, out)
        torch.cuda.synchronize()
        vals.append(float(out.item()))
    assert abs(vals[0] - vals[1]) <= 1e-12 * abs(vals[0])


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("threads", [64, 256, 512])
@pytest.mark.parametrize("lds", [163840, 20480])
def test_split_products(dtype, threads, lds):
    """Few blocks and long sums: K in ranges over the workgroup's waves (the
    last one short or empty), whose results are added in LDS."""
    rng = np.random.default_rng(threads + lds)
    for m, n, k in [(4, 6, 3456), (16, 16, 2049), (15, 17, 257), (33, 16, 128), (64, 13, 131), (16, 48, 130),
                    (5, 7, 1000), (17, 17, 129)]:
        a = rng.uniform(-1, 1, (k, m)).astype(dtype).astype(np.float64)
        b = rng.uniform(-1, 1, (k, n)).astype(dtype).astype(np.float64)
        got = _run([a, b], [[0, 1], [0, 2]], [k, m, n], [1, 2], dtype, threads, lds).reshape(m, n)
        bound = 2 * (k + 2) * U[dtype] * (np.abs(a).T @ np.abs(b))
        assert (np.abs(got - a.T @ b) <= bound).all(), (m, n, k)
