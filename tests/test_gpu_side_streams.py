"""Clocks and streams of batches that mix fused networks with networks on side
streams."""

import numpy as np
import pytest

from paper_2410_15080_amd import htn
from workloads import configs
from workloads.network import Network

from gpu_helpers import create
from test_gpu_level_dispatch import _products

pytestmark = pytest.mark.gpu


def _run(b, outs, stream):
    import torch
    with torch.cuda.stream(stream):
        htn.htn_batch_run(b, htn.pointer_array(outs), stream)
    stream.synchronize()


@pytest.mark.parametrize("fused", [0, 96])
@pytest.mark.parametrize("how", ["eager", "graph", "phases"])
def test_the_run_starts_before_its_networks(how, fused):
    """Fused networks (with inputs to materialise), queued ones where there are
    no fused ones, and one network with a launch per step: no clock of the run
    lies before its start (but for the tick that two XCDs' clocks may differ)."""
    import torch
    nets = [create(configs.grid_network(s)) for s in range(fused or 2)]
    if not fused:
        for n in nets:
            htn.htn_set_option(n, htn.HTN_OPT_QUEUE, 1)
    step, _ = _products(1)
    htn.htn_set_option(step[0], htn.HTN_OPT_QUEUE, 2)
    nets += step
    outs = [htn.new_output(n) for n in nets]
    b = htn.htn_batch_create(nets)
    assert htn.htn_batch_level_info(b)[0] == 0
    if how == "phases":
        htn.htn_batch_set_phase_timing(b, 4)
    htn.htn_batch_set_graph(b, how == "graph")
    stream = torch.cuda.Stream()
    for rep in range(40):
        _run(b, outs, stream)
        t = htn.htn_batch_timestamps(b)
        assert (t[:, 0] >= -1).all() and (t[:, 1] >= t[:, 0]).all(), (rep, t.min())
        if how == "phases":
            assert (htn.htn_batch_phase_times(b) >= -1).all(), rep
    htn.htn_batch_destroy(b)


def _chain(seed, n=40, d=90):
    """A product of n small matrices, from the first to the last."""
    rng = np.random.default_rng(seed)
    path, at = [], 0
    for k in range(1, n):
        path.append((at, k))
        at = n + k - 1
    return create(Network([rng.uniform(-0.1, 0.1, size=(d, d)) for _ in range(n)], [[k, k + 1] for k in range(n)],
                          [d] * (n + 1), [0, n]), exec_mode=htn.HTN_EXEC_STEPS, path=path)


def test_heavy_network_does_not_wait_for_the_levels():
    """A network above the level launches' size limit runs beside them (39 small
    steps in a row, which leave the chip idle), on a stream of its own, though
    it is the heaviest.  As a graph: eager launches reach the device one by one."""
    import torch
    big, refs = _products(1, 1100, 1000, 1000)  # more than 2^30 multiplications
    nets = big + [_chain(0), _chain(1)]
    outs = [htn.new_output(n) for n in nets]
    b = htn.htn_batch_create(nets)
    info = htn.htn_batch_level_info(b)
    assert info[0] == 2 and info[1] >= 39 and htn.htn_batch_queue_info(b)[0] == 0, info
    htn.htn_batch_set_graph(b, True)
    stream = torch.cuda.Stream()
    _run(b, outs, stream)
    assert htn.htn_batch_graph_state(b) == 1
    starts, ends = [], []
    for _ in range(5):
        _run(b, outs, stream)
        t = htn.htn_batch_timestamps(b)
        starts.append(t[0, 0])
        ends.append(t[1:, 1].max())
    assert np.array_equal(outs[0].cpu().numpy().reshape(refs[0].shape), refs[0])
    assert np.median(starts) < np.median(ends), (starts, ends)
    htn.htn_batch_destroy(b)


def test_fused_networks_do_not_wait_for_the_levels_to_be_launched():
    """Eager: the fused launch is issued ahead of the 40 level launches, each of
    which takes the host some microseconds."""
    import torch
    nets = [create(configs.grid_network(s), lds=81920) for s in range(256)] + [_chain(0), _chain(1)]
    outs = [htn.new_output(n) for n in nets]
    b = htn.htn_batch_create(nets)
    assert htn.htn_batch_level_info(b)[0] == 2
    stream = torch.cuda.Stream()
    waits = []
    for _ in range(6):
        _run(b, outs, stream)
        t = htn.htn_batch_timestamps(b)
        waits.append(np.median(t[:256, 0]) / t[256:, 1].max())
    assert np.median(waits) < 0.5, waits
    htn.htn_batch_destroy(b)
