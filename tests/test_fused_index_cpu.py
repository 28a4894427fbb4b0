"""The fused program's index against the program itself: every phase's
copies, and for each wave the step it runs, are where the index says."""

import json

import numpy as np
import pytest

from paper_2410_15080_amd import htn
from tests.plan_emulator import OP_COPY, OP_END, OP_STEP, OP_SYNC, OP_TSTEP
from workloads import configs


def _walk(prog):
    """[(copy offsets, [(step offset, op words)])] per phase, in program order."""
    p, phases, copies, steps = 8, [], [], []
    while prog[p] != OP_END:
        op = prog[p]
        if op == OP_SYNC:
            phases.append((copies, steps))
            copies, steps = [], []
            p += 1
        elif op == OP_COPY:
            assert not steps, "a phase lists its copies first"
            copies.append(p)
            p += 5
        else:
            n = 15 + 4 * (prog[p + 11] + prog[p + 12]) if op == OP_TSTEP else 17
            assert op in (OP_STEP, OP_TSTEP)
            steps.append((p, prog[p:p + n]))
            p += n
    assert not copies and not steps
    return phases, p


@pytest.mark.parametrize("threads", [64, 256, 512])
@pytest.mark.parametrize("make", [lambda: configs.grid_network(3), lambda: configs.grid_network(5, 2, 2),
                                  lambda: configs.ring_of_rings(1, 4, 6),
                                  lambda: configs.random_network(np.random.default_rng([7, 3]))])
@pytest.mark.parametrize("tight", [False, True])
def test_index_matches_program(make, threads, tight):
    """tight: the smallest LDS budget that takes the program without its index."""
    w = make()
    net = htn.htn_create([np.asarray(t, dtype=np.float64) for t in w.tensors], w.labels, w.dims, w.out_labels)
    htn.htn_set_option(net, htn.HTN_OPT_FUSED_THREADS, threads)
    prog = json.loads(htn.htn_plan_json(net))["program"]
    W = threads // 64
    if tight:
        words = prog[0] - (1 + len(_walk(prog)[0]) * (2 + W))
        htn.htn_set_option(net, htn.HTN_OPT_FUSED_LDS_BYTES, max(1024, ((words + 3) // 4 * 4 + 2 * prog[4]) * 4 + 256))
        prog = json.loads(htn.htn_plan_json(net))["program"]
    phases, end = _walk(prog)
    at = prog[2]
    assert end < at and (at + 1 + len(phases) * (2 + W) <= prog[0] or at >= prog[0])

    assert prog[at] == len(phases)
    for k, (copies, steps) in enumerate(phases):
        e = prog[at + 1 + k * (2 + W):at + 1 + (k + 1) * (2 + W)]
        assert e[1] == len(copies)
        if copies:
            assert e[0] == copies[0] and copies == list(range(e[0], e[0] + 5 * e[1], 5))
        for wave in range(W):
            want = 0
            for off, words in steps:
                w0, nw = (words[13], words[14]) if words[0] == OP_TSTEP else (words[15], words[16])
                if w0 <= wave < w0 + nw:
                    want = off
                    if words[0] == OP_TSTEP and words[7] == 0:  # 16x16 blocks: idle waves have none
                        blocks = -(-words[4] // 16) * -(-words[5] // 16)
                        want = off if wave - w0 < blocks else 0
            assert e[2 + wave] == want
