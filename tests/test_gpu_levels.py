"""Level launches of a batch: the steps of all its step-by-step networks,
one launch per dependency level.

They run the per-step kernels' own bodies on the same plan, so every network
must come out bit for bit equal to its per-step launches."""

import numpy as np
import pytest

from paper_2410_15080_amd import htn
from workloads import configs

from gpu_helpers import create
from test_gpu_queue import _fs, _run_batch, _workloads

pytestmark = pytest.mark.gpu


def _heavy(compute):
    """Networks that neither the queue nor the fused kernel takes by default:
    ragged matrix products (with a batch label, with a split sum), long split
    sums, and random networks with scaled inputs."""
    ws = _workloads("gemm") + _workloads("split_sum")
    rnd = configs.random_batch(0, n=320, dtype=np.float64)
    return ws + [rnd[i] for i in (18, 44, 109, 251, 281, 297)]


@pytest.mark.parametrize("compute", [htn.HTN_F64, htn.HTN_F32, htn.HTN_BF16])
def test_levels_match_per_step_launches_bit_for_bit(compute):
    """Also over graph replays, with the caller's work between them, and with
    a start and an end clock for every network."""
    import torch
    ws = _heavy(compute)
    made = [[create(w, compute=compute, final_sum=_fs(compute), storage=htn.HTN_F64, exec_mode=htn.HTN_EXEC_STEPS)
             for w in ws] for _ in range(2)]
    for n in made[1]:
        htn.htn_set_option(n, htn.HTN_OPT_QUEUE, 2)
    outs = [[htn.new_output(n) for n in nets] for nets in made]
    bl, rl = _run_batch(made[0], outs[0])
    bs, rs = _run_batch(made[1], outs[1])
    assert htn.htn_batch_queue_info(bl)[:2] == (0, 0)
    for i, (a, b) in enumerate(zip(rl[0], rs[0])):
        assert np.isfinite(a).all() and np.array_equal(a, b), i
    htn.htn_batch_set_graph(bl, True)
    stream = torch.cuda.Stream()
    for rep in range(3):
        for o in outs[0]:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            htn.htn_batch_run(bl, htn.pointer_array(outs[0]), stream)
        stream.synchronize()
        x = torch.zeros(1 << 20, device="cuda")
        x.add_(1.0)
        torch.cuda.synchronize()
        for i, o in enumerate(outs[0]):
            assert np.array_equal(o.cpu().numpy(), rs[0][i]), (rep, i)
        t = htn.htn_batch_timestamps(bl)
        assert (t[:, 1] > t[:, 0]).all() and (t[:, 0] >= -1).all(), rep
    htn.htn_batch_destroy(bl)
    htn.htn_batch_destroy(bs)
