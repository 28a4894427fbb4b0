"""The final product in either output order, with the final sum that was asked
for.

C[n, m] = sum_k A[m, k] B[k, n] read N first is the same matrix product with
its operands exchanged; htn_final_sum promises the last step's products and
sums in FP64 (HTN_SUM_FP64) or compensated (HTN_SUM_COMPENSATED) whatever the
order, and a folded operand in FP32 until then.  Bounds are those of the
arithmetic: K roundings of the accumulator per sum, against long double or
exact integers."""

import json

import numpy as np
import pytest

from paper_2410_15080_amd import htn
from workloads.network import Network

COMPUTE = [htn.HTN_F64, htn.HTN_F32, htn.HTN_BF16]
EPS = {htn.HTN_F64: 2.0 ** -53, htn.HTN_F32: 2.0 ** -24, htn.HTN_BF16: 2.0 ** -24}
# (M, N, K): both sides of the bound above which operands are packed (2^25
# multiplications), ragged tiles, K split into ranges and with a short last chunk
SHAPES = [(300, 420, 48), (700, 900, 64), (333, 4001, 33), (64, 72, 4100)]


def _rounded(x, compute):
    """x in the compute type's input format, as FP64."""
    if compute == htn.HTN_F64:
        return np.asarray(x, dtype=np.float64)
    import torch
    t = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64))
    return t.to(torch.float32 if compute == htn.HTN_F32 else torch.bfloat16).to(torch.float64).numpy()


def _product(rng, M, N, K, n_first, compute=htn.HTN_F64):
    a, b = (_rounded(rng.standard_normal(s), compute) for s in ((M, K), (K, N)))
    return Network([a, b], [[0, 2], [2, 1]], [M, N, K], [1, 0] if n_first else [0, 1])


def _last(w, compute, final_sum, exec_mode=htn.HTN_EXEC_AUTO):
    net = htn.htn_create(w.tensors, w.labels, w.dims, w.out_labels, compute=compute, final_sum=final_sum,
                         storage=htn.HTN_F64)
    htn.htn_set_option(net, htn.HTN_OPT_EXEC, exec_mode)
    return json.loads(htn.htn_plan_json(net))["steps"][-1]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("compute", COMPUTE)
def test_exchanged_product_keeps_its_arithmetic(shape, compute):
    """No packing (which rounds to BF16, and whose FP32 chunks are not FP64
    sums) for an FP32 or BF16 product read N first, and no matrix instructions
    for compensated sums."""
    w = _product(np.random.default_rng(1), *shape, True)
    for final_sum in (htn.HTN_SUM_PLAIN, htn.HTN_SUM_FP64):
        s = _last(w, compute, final_sum)
        assert s["mfma"] and (compute == htn.HTN_F64 or s["xtile"][0]), final_sum
    s = _last(w, compute, htn.HTN_SUM_COMPENSATED)
    assert not s["mfma"] and not s["xtile"][0]


def _contract(w, compute, final_sum, exec_mode, path=None, tiled=True):
    import torch
    ts = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda") for t in w.tensors]
    net = htn.htn_create(ts, w.labels, w.dims, w.out_labels, compute=compute, final_sum=final_sum,
                         storage=htn.HTN_F64)
    if path is not None:  # the last step is the exchanged product
        htn.htn_set_path(net, path)
        assert json.loads(htn.htn_plan_json(net))["steps"][-1]["xtile"][0] == tiled
    htn.htn_set_option(net, htn.HTN_OPT_EXEC, exec_mode)
    out = htn.new_output(net)
    htn.htn_contract(net, out)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64).reshape([w.dims[l] for l in w.out_labels])


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("compute", COMPUTE)
def test_final_sum_error(shape, compute):
    """Inputs whose products and sums all round."""
    M, N, K = shape
    w = _product(np.random.default_rng(K), M, N, K, True, compute)
    a, b = w.tensors
    ref = (a.astype(np.longdouble) @ b.astype(np.longdouble)).T
    mag = (np.abs(a) @ np.abs(b)).T
    for final_sum in (htn.HTN_SUM_PLAIN, htn.HTN_SUM_FP64, htn.HTN_SUM_COMPENSATED):
        eps = EPS[compute] if final_sum == htn.HTN_SUM_PLAIN else 2.0 ** -53
        for mode in (htn.HTN_EXEC_AUTO, htn.HTN_EXEC_STEPS):
            got = _contract(w, compute, final_sum, mode)
            err = np.abs(got - ref) / mag
            assert err.max() <= (K + 2) * eps, (final_sum, mode, float(err.max()))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,W,tiled", [(1100, 64, 16, True), (2100, 32, 32, True), (1100, 64, 64, False)])
@pytest.mark.parametrize("compute", [htn.HTN_F32, htn.HTN_BF16])
def test_folded_operand_is_not_rounded(M, K, W, tiled, compute):
    """One operand is a step's FP32 result (a plain step's, a fold chain's, and
    a packed product's, whose layout is its own, so that no exchange follows):
    its own sums' error and no more."""
    rng = np.random.default_rng(W)
    N = 1500
    t1, v, t2 = (_rounded(rng.standard_normal(s), compute) for s in ((W, M), (W, K), (K, N)))
    w = Network([t1, v, t2], [[3, 0], [3, 2], [2, 1]], [M, N, K, W], [1, 0])
    fold = t1.T.astype(np.longdouble) @ v.astype(np.longdouble)
    ref = (fold @ t2.astype(np.longdouble)).T
    mag = ((np.abs(t1).T @ np.abs(v)) @ np.abs(t2)).T
    for final_sum, eps in ((htn.HTN_SUM_PLAIN, 2.0 ** -24), (htn.HTN_SUM_FP64, 2.0 ** -53)):
        got = _contract(w, compute, final_sum, htn.HTN_EXEC_AUTO, path=[(0, 1), (3, 2)], tiled=tiled)
        err = np.abs(got - ref) / mag
        assert err.max() <= (W + 1) * 2.0 ** -24 + (K + 2) * eps, (final_sum, float(err.max()))


@pytest.mark.gpu
@pytest.mark.parametrize("compute", COMPUTE)
def test_compensated_sums_stay_compensated(compute):
    """Exact products of both signs that cancel to a few of their last bits:
    the compensated sum keeps them (an error of 2^-53 of the sum, and of
    2^-106 of the terms per addition), a plain FP64 one does not."""
    rng = np.random.default_rng(9)
    M, N, H = 300, 420, 24
    bits = {htn.HTN_F64: 25, htn.HTN_F32: 22, htn.HTN_BF16: 6}[compute]
    a = rng.integers(-2 ** bits, 2 ** bits, size=(M, H))
    b = rng.integers(1, 2 ** bits, size=(H, N))
    d = rng.integers(-3, 4, size=(M, H))
    e = 2 ** rng.integers(0, 28, size=H)
    w = Network([np.concatenate([a * e, (d - a) * e], axis=1).astype(np.float64),
                 np.concatenate([b, b], axis=0).astype(np.float64)], [[0, 2], [2, 1]], [M, N, 2 * H], [1, 0])
    ref = ((d * e).astype(object) @ b.astype(object)).T
    mag = 2 * ((np.abs(a) + 3) * e).astype(np.float64) @ b.astype(np.float64)
    got = _contract(w, compute, htn.HTN_SUM_COMPENSATED, htn.HTN_EXEC_AUTO)
    err = np.array([[abs(int(x) - int(y)) for x, y in zip(r, s)] for r, s in zip(got, ref)], dtype=np.float64)
    bound = 2 * (2.0 ** -53 * np.abs(ref.astype(np.float64)) + (2 * H) ** 2 * 2.0 ** -106 * mag.T)
    assert (err <= bound).all(), float((err / np.maximum(bound, 1e-300)).max())


@pytest.mark.parametrize("shape", SHAPES)
def test_executor_choice_leaves_the_plan(shape):
    w = _product(np.random.default_rng(2), *shape, True)
    net = htn.htn_create(w.tensors, w.labels, w.dims, w.out_labels, final_sum=htn.HTN_SUM_FP64)
    plan = htn.htn_plan_json(net)
    for mode in (htn.HTN_EXEC_FUSED, htn.HTN_EXEC_STEPS, htn.HTN_EXEC_AUTO):
        htn.htn_set_option(net, htn.HTN_OPT_EXEC, mode)
        assert htn.htn_plan_json(net) == plan, mode


@pytest.mark.gpu
@pytest.mark.parametrize("compute", COMPUTE)
def test_batch_outlives_a_change_of_executor(compute):
    """A batch runs as it was made; the fused kernel, asked for, takes the same
    plan (small whole numbers: every sum is exact)."""
    import torch
    rng = np.random.default_rng(3)
    ws = [Network([rng.integers(-8, 9, size=(M, K)).astype(np.float64), rng.integers(-8, 9, size=(K, N)).astype(np.float64)],
                  [[0, 2], [2, 1]], [M, N, K], [1, 0]) for M, N, K in SHAPES]
    refs = [(w.tensors[0] @ w.tensors[1]).T for w in ws]
    ts = [[torch.from_numpy(t).to("cuda") for t in w.tensors] for w in ws]
    nets = [htn.htn_create(t, w.labels, w.dims, w.out_labels, compute=compute, final_sum=htn.HTN_SUM_FP64,
                           storage=htn.HTN_F64) for t, w in zip(ts, ws)]
    outs = [htn.new_output(n) for n in nets]
    b = htn.htn_batch_create(nets)
    for mode in (htn.HTN_EXEC_AUTO, htn.HTN_EXEC_FUSED, htn.HTN_EXEC_STEPS):
        for n, o, ref in zip(nets, outs, refs):
            htn.htn_set_option(n, htn.HTN_OPT_EXEC, mode)
            htn.htn_contract(n, o)
            torch.cuda.synchronize()
            assert np.array_equal(o.cpu().numpy().reshape(ref.shape), ref), (mode, ref.shape)
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        htn.htn_batch_run(b, htn.pointer_array(outs))
        torch.cuda.synchronize()
        for o, ref in zip(outs, refs):
            assert np.array_equal(o.cpu().numpy().reshape(ref.shape), ref), (mode, ref.shape)
    htn.htn_batch_destroy(b)


@pytest.mark.gpu
@pytest.mark.parametrize("compute", COMPUTE)
def test_queue_levels_and_launches_agree(compute):
    """The exchanged product as a queue's and a level's item and as launches,
    K ranges included: the same bits, within the bound of FP64 sums."""
    import torch
    rng = np.random.default_rng(12)
    ws = [_product(rng, *s, True, compute) for s in SHAPES]
    ts = [[torch.from_numpy(t).to("cuda") for t in w.tensors] for w in ws]
    runs = []
    for queue in (0, 1, 2):
        nets = [htn.htn_create(t, w.labels, w.dims, w.out_labels, compute=compute, final_sum=htn.HTN_SUM_FP64,
                               storage=htn.HTN_F64) for t, w in zip(ts, ws)]
        for n in nets:
            htn.htn_set_option(n, htn.HTN_OPT_EXEC, htn.HTN_EXEC_STEPS)
            htn.htn_set_option(n, htn.HTN_OPT_QUEUE, queue)
        outs = [htn.new_output(n) for n in nets]
        b = htn.htn_batch_create(nets)
        assert htn.htn_batch_queue_info(b)[0] == (len(nets) if queue == 1 else 0)
        assert htn.htn_batch_level_info(b)[0] == (len(nets) if queue == 0 else 0)
        htn.htn_batch_run(b, htn.pointer_array(outs))
        torch.cuda.synchronize()
        runs.append([o.cpu().numpy() for o in outs])
        htn.htn_batch_destroy(b)
    for k, (w, (M, N, K)) in enumerate(zip(ws, SHAPES)):
        assert np.array_equal(runs[0][k], runs[1][k]) and np.array_equal(runs[0][k], runs[2][k]), k
        a, b = w.tensors
        ref, mag = (a.astype(np.longdouble) @ b.astype(np.longdouble)).T, (np.abs(a) @ np.abs(b)).T
        assert (np.abs(runs[0][k].reshape(ref.shape) - ref) <= (K + 2) * 2.0 ** -53 * mag).all(), k
