"""Which networks of a batch run in the level launches, and the block-to-item
search of levels of many items."""

import json

import numpy as np
import pytest

from paper_2410_15080_amd import htn
from workloads.network import Network

from gpu_helpers import create
from test_gpu_levels import _heavy
from test_gpu_queue import _fs, _run_batch

pytestmark = pytest.mark.gpu


def _products(n, M=90, N=84, K=80):
    """n products of small whole numbers (exact in every type) on shared device
    tensors, A[i] B[j]; kernel steps too large for the queue by default, too
    small for a matrix product of their own."""
    import torch
    rng = np.random.default_rng(n)
    a = [rng.integers(-8, 9, size=(M, K)).astype(np.float64) for _ in range(7)]
    b = [rng.integers(-8, 9, size=(K, N)).astype(np.float64) for _ in range(5)]
    ta, tb = ([torch.from_numpy(x).to("cuda") for x in xs] for xs in (a, b))
    nets = []
    for k in range(n):
        net = htn.htn_create([ta[k % 7], tb[k % 5]], [[0, 2], [2, 1]], [M, N, K], [0, 1])
        htn.htn_set_option(net, htn.HTN_OPT_EXEC, htn.HTN_EXEC_STEPS)
        nets.append(net)
    refs = {(i, j): a[i] @ b[j] for i in range(7) for j in range(5)}
    return nets, [refs[k % 7, k % 5] for k in range(n)]


# one step of the search covers 64 items, two 4096
@pytest.mark.parametrize("n", [2, 64, 65, 4097])
def test_levels_of_many_items(n):
    nets, refs = _products(n)
    outs = [htn.new_output(x) for x in nets]
    b, r = _run_batch(nets, outs)
    assert htn.htn_batch_queue_info(b)[:2] == (0, 0)
    assert htn.htn_batch_level_info(b)[0] == n and htn.htn_batch_level_info(b)[2] >= n
    for k, (got, ref) in enumerate(zip(r[0], refs)):
        assert np.array_equal(got.reshape(ref.shape), ref), k
    htn.htn_batch_destroy(b)


def _expected(nets):
    """Networks of one kind of packed product (into FP64 or not) share the
    launches, that of the heaviest one with such a product; those without
    any join them."""
    kind, n = None, 0
    for net in sorted(nets, key=lambda x: -htn.htn_get_info(x).mults):
        steps = json.loads(htn.htn_plan_json(net))["steps"]
        kinds = {k == len(steps) - 1 and net.compute != htn.HTN_F64 for k, s in enumerate(steps)
                 if s["mfma"] and not s["xtile"][0]}
        if len(kinds) > 1 or (kinds and kind is not None and kinds != kind):
            continue
        kind = kinds or kind
        n += 1
    return n


@pytest.mark.parametrize("compute", [htn.HTN_F64, htn.HTN_F32, htn.HTN_BF16])
def test_networks_that_take_level_launches(compute):
    """The networks compared with launches per step elsewhere run in levels (in
    FP64 all of them); with an option they stay out, and one alone does."""
    ws = _heavy(compute)
    nets = [create(w, compute=compute, final_sum=_fs(compute), storage=htn.HTN_F64, exec_mode=htn.HTN_EXEC_STEPS)
            for w in ws]
    for n in nets:
        n.compute = compute
    expected = _expected(nets)
    assert expected == len(ws) or compute != htn.HTN_F64
    for queue, expected in ((0, expected), (2, 0)):
        for n in nets:
            htn.htn_set_option(n, htn.HTN_OPT_QUEUE, queue)
        b = htn.htn_batch_create(nets)
        got = htn.htn_batch_level_info(b)
        assert got[0] == expected and (got[1] >= 2) == (expected > 0), (queue, got)
        htn.htn_batch_destroy(b)
    htn.htn_set_option(nets[0], htn.HTN_OPT_QUEUE, 0)
    b = htn.htn_batch_create(nets)
    assert htn.htn_batch_level_info(b) == (0, 0, 0)
    htn.htn_batch_destroy(b)


def test_mixed_batch_keeps_one_network_out():
    """A network of fold chains has a kernel of its own: it runs beside the
    level launches, with one launch per step."""
    rng = np.random.default_rng(4)
    c = [rng.integers(-2, 3, size=(4, 4)).astype(np.float64) for _ in range(2)]
    t1, t2 = rng.integers(-2, 3, size=(4, 4, 4200)), rng.integers(-2, 3, size=(4, 4, 80))
    w = Network([t1.astype(np.float64), t2.astype(np.float64), *c], [[0, 1, 4], [2, 3, 5], [0, 2], [1, 3]],
                [4, 4, 4, 4, 4200, 80], [4, 5])
    ref = np.einsum("abm,cdn,ac,bd->mn", t1, t2, *c, optimize=True)
    out = create(w, exec_mode=htn.HTN_EXEC_STEPS, path=[(0, 2), (4, 3), (5, 1)])
    htn.htn_set_option(out, htn.HTN_OPT_QUEUE, 0)
    nets, refs = _products(3)
    nets.append(out)
    outs = [htn.new_output(n) for n in nets]
    b, r = _run_batch(nets, outs)
    n_level = htn.htn_batch_level_info(b)[0]
    n_queue = htn.htn_batch_queue_info(b)[0]
    assert (n_level, n_queue) == (3, 0), (n_level, n_queue)
    for got, want in zip(r[0], refs + [ref]):
        assert np.array_equal(got.reshape(want.shape), want)
    htn.htn_batch_destroy(b)


def test_level_launches_use_the_callers_allocator():
    """The launches' intermediates and lists come from the caller's allocator
    and go back to it; where it has none, the networks run with a launch per
    step as before, with the same results."""
    import torch
    ws = _heavy(htn.HTN_F64)
    nets = [create(w, final_sum=htn.HTN_SUM_COMPENSATED, exec_mode=htn.HTN_EXEC_STEPS) for w in ws]
    outs = [htn.new_output(n) for n in nets]
    b, ref = _run_batch(nets, outs)  # (the nets' own buffers are made here)
    assert htn.htn_batch_level_info(b)[0] == len(nets)
    htn.htn_batch_destroy(b)
    held, sizes, limit = {}, [], [None]

    def alloc(n):
        if limit[0] is not None and n > limit[0]:
            return 0
        t = torch.empty(n, dtype=torch.uint8, device="cuda")
        held[t.data_ptr()] = t
        sizes.append(n)
        return t.data_ptr()

    htn.htn_set_allocator(alloc, lambda p: held.pop(p, None))
    try:
        for cap in (None, 1 << 20, 1 << 13):
            limit[0] = cap
            del sizes[:]
            b, r = _run_batch(nets, outs)
            n = htn.htn_batch_level_info(b)[0]
            assert n == (len(nets) if cap is None else 0), cap
            assert cap is not None or max(sizes) > 1 << 20
            assert all(np.array_equal(x, y) for x, y in zip(r[0], ref[0])), cap
            htn.htn_batch_destroy(b)
            assert not held, cap
    finally:
        torch.cuda.synchronize()
        htn.htn_set_allocator(None, None)
