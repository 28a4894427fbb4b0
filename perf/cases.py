"""The performance cases: hybrid-tensor-network (h-TN) contraction as a user's
program has it done, through the public entry points of paper_2410_15080_amd.

Families (case["family"]):
  circuit    a cut circuit end to end: the QT evaluator simulates every
             subcircuit instance and assembles the QTs, then the network is
             contracted (one network, one htn_contract).
  single     one network whose QTs are already tensors, contracted by itself.
  batch      many independent networks contracted by one reusable batch, as
             eager launches or as a replayed graph.
  qpd        the batch after QPD sampling: one step truncates every QT to its
             drawn terms and contracts the simplified networks.
  marginal   one network with open outputs: two QTs [4]*n_cuts + [outputs]
             joined by CutQC wire tensors.
  model      the path cost model: predictions and the gradients of a training
             step.

A case fixes the structure (labels, extents, circuits' shapes); the seed of
prepare() gives the values.
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2410_15080_amd import htn
from paper_2410_15080_amd import qpd as htn_qpd
from paper_2410_15080_amd import qteval
from workloads import circuits, configs
from workloads import qpd as coeffs

COMPUTE = {"f64": htn.HTN_F64, "f32": htn.HTN_F32, "bf16": htn.HTN_BF16}
TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"f64": 8, "f32": 4, "bf16": 2}
FINAL = {"plain": htn.HTN_SUM_PLAIN, "fp64": htn.HTN_SUM_FP64, "compensated": htn.HTN_SUM_COMPENSATED}


def listed():
    return [
        # The smallest whole call: the 10-qubit circuit with two wire cuts,
        # 44 instances of 3 to 5 qubits, evaluated and contracted.  Launches
        # and latency are all of it.
        {"name": "circuit10", "family": "circuit", "kind": "wires", "first": 0},
        # Subcircuits of the largest size of the workloads (15 qubits), both
        # sides keeping 6 qubits: 80 instances, a 64 x 64 marginal.
        {"name": "circuit_marginal15", "family": "circuit", "kind": "marginal", "first": 0, "n_left": 15,
         "n_right": 15, "cuts": 2, "layers": 4, "kept": 6},
        # One 4x4 grid h-TN by itself, as an interactive program asks for one
        # expectation value.
        {"name": "grid_one_f64", "family": "single", "net": "grid", "rows": 4, "cols": 4, "first": 0,
         "dtype": "f64", "final": "plain", "samples": 32},
        # The headline workload: 1024 4x4 grids of wire and CZ cuts, replayed
        # as a graph on sampled paths.
        {"name": "grid1024_f64", "family": "batch", "net": "grid", "rows": 4, "cols": 4, "first": 0, "nets": 1024,
         "dtype": "f64", "final": "plain", "samples": 32, "threads": 256, "lds": 81920, "graph": True},
        # The same grids after drawing every gate cut 8 times (few samples a
        # cut): the truncation gather and the contraction, step by step.
        {"name": "qpd1024_f64", "family": "qpd", "rows": 4, "cols": 4, "first": 0, "nets": 1024, "draws": 8,
         "dtype": "f64", "samples": 32, "threads": 256, "lds": 81920},
        # Networks of 64 QTs (eight rings of eight), the largest that a batch
        # is made of, with the compensated final sum.
        {"name": "ring256_f64", "family": "batch", "net": "ring", "rings": 8, "length": 8, "first": 0, "nets": 256,
         "dtype": "f64", "final": "compensated", "samples": 0, "threads": 512, "lds": 163840, "graph": True},
        # A smaller batch of smaller rings with BF16 inputs, at the library's
        # default workgroup and LDS budget, one eager run.
        {"name": "ring60_bf16", "family": "batch", "net": "ring", "rings": 6, "length": 8, "first": 1000, "nets": 60,
         "dtype": "bf16", "final": "plain", "samples": 0, "threads": 256, "lds": 65536, "graph": False},
        # A serving batch of uneven random networks (3 to 12 QTs, 2 to 14
        # cuts), FP32.
        {"name": "random512_f32", "family": "batch", "net": "random", "first": 0, "nets": 512, "dtype": "f32",
         "final": "plain", "samples": 0, "threads": 512, "lds": 163840, "graph": True},
        # The 4096 x 4096 marginal of two QTs joined by four wire cuts.
        {"name": "marginal4096_f64", "family": "marginal", "left": 4096, "right": 4096, "cuts": 4, "dtype": "f64",
         "final": "fp64"},
        {"name": "marginal4096_bf16", "family": "marginal", "left": 4096, "right": 4096, "cuts": 4, "dtype": "bf16",
         "final": "fp64"},
        # Outputs that are no power of two (a post-selected set of bitstrings
        # on either side) and three cuts, FP32.
        {"name": "marginal_ragged_f32", "family": "marginal", "left": 2999, "right": 1531, "cuts": 3, "dtype": "f32",
         "final": "fp64"},
        # One step of the cost model over a training set's size of steps.
        {"name": "model_step", "family": "model", "rows": 14227},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    fam = rng.choice(["circuit", "single", "batch", "batch", "qpd", "marginal", "marginal", "model"])
    first = 2000 + 1000 * rng.randrange(1000)
    if fam == "circuit":
        left, right, cuts = rng.randint(5, 15), rng.randint(5, 15), rng.randint(1, 2)
        return {"family": "circuit", "kind": "marginal", "first": first, "n_left": left, "n_right": right,
                "cuts": cuts, "layers": rng.randint(2, 4), "kept": rng.randint(1, min(6, left - cuts, right - cuts))}
    if fam == "single":
        return {"family": "single", "net": "grid", "rows": rng.randint(2, 4), "cols": rng.randint(2, 5),
                "first": first, "dtype": rng.choice(["f64", "f32"]), "final": "plain", "samples": 32}
    if fam == "batch":
        threads, lds = rng.choice([(256, 65536), (256, 81920), (512, 163840)])
        c = {"family": "batch", "first": first, "threads": threads, "lds": lds, "graph": rng.random() < 0.5}
        dtype = rng.choice(["f64", "f64", "f32", "bf16"])
        c["dtype"] = dtype
        c["final"] = rng.choice(["plain", "compensated"]) if dtype == "f64" else "plain"
        net = rng.choice(["grid", "grid", "ring", "random"])
        c["net"] = net
        if net == "grid":
            c.update(rows=rng.randint(2, 4), cols=rng.randint(2, 4), nets=_log_int(rng, 3, 700), samples=32)
        elif net == "ring":
            c.update(rings=rng.randint(3, 8), length=rng.choice([6, 7, 8]), nets=_log_int(rng, 3, 200), samples=0)
        else:
            c.update(nets=_log_int(rng, 3, 256), samples=0)
        return c
    if fam == "qpd":
        return {"family": "qpd", "rows": rng.randint(2, 4), "cols": rng.randint(2, 4), "first": first,
                "nets": _log_int(rng, 3, 700), "draws": rng.choice([1, 2, 4, 8, 16, 64]), "dtype": "f64",
                "samples": 32, "threads": 256, "lds": rng.choice([65536, 81920])}
    if fam == "marginal":
        return {"family": "marginal", "left": _log_int(rng, 16, 4096), "right": _log_int(rng, 16, 4096),
                "cuts": rng.randint(1, 4), "dtype": rng.choice(["f64", "f32", "bf16"]), "final": "fp64"}
    return {"family": "model", "rows": _log_int(rng, 64, 14227)}


# ------------------------------------------------------------- structures

@functools.lru_cache(maxsize=64)
def _structures(key):
    """(labels, dims, kinds) per network of a batch: what a case fixes."""
    c = dict(key)
    out = []
    for i in range(c.get("nets", 1)):
        s = c["first"] + i
        if c["net"] == "grid":
            w = configs.grid_network(s, c["rows"], c["cols"])
        elif c["net"] == "ring":
            w = configs.ring_of_rings(s, c["rings"], c["length"])
        else:
            w = configs.random_network(np.random.default_rng([c["first"], i]))
        out.append((w.labels, w.dims, w.kinds))
    return out


def _key(case):
    keys = ("net", "rows", "cols", "rings", "length", "first", "nets")
    c = dict(case, net=case.get("net", "grid"))
    if case["family"] == "single":
        c["nets"] = 1
    return tuple((k, c[k]) for k in keys if k in c)


def _nets_of(case):
    return _structures(_key(case))


@functools.lru_cache(maxsize=64)
def _paths(key, samples):
    """The contraction paths of a batch's structures, searched once as a
    program that meets the same circuits again does (the values and the
    drawn terms change, the search is kept)."""
    out = []
    for labels, dims, _ in _structures(key):
        net = htn.htn_create([np.zeros([dims[l] for l in ls]) for ls in labels], labels, dims)
        htn.htn_set_option(net, htn.HTN_OPT_PATH_SAMPLES, samples)
        htn.htn_set_path(net, htn.HTN_PATH_SAMPLED)
        out.append(htn.htn_get_path(net)[0])
    return out


def _ct(dim):
    return coeffs.WIRE_PAULI if dim == 4 else coeffs.CZ_COEFFS


def _values(case, seed):
    """Per network its tensors on the GPU: QT entries U[-1, 1], the cuts'
    QPD weights."""
    dt = TORCH[case["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    vecs = {d: torch.from_numpy(_ct(d).copy()).to("cuda", dt) for d in (4, 6)}
    nets = _nets_of(case)
    sizes = [[math.prod(dims[l] for l in ls) for ls in labels] for labels, dims, _ in nets]
    pool = torch.rand(sum(map(sum, sizes)), generator=gen, device="cuda", dtype=torch.float64)
    pool = (2.0 * pool - 1.0).to(dt)
    out, at = [], 0
    for (labels, dims, kinds), sz in zip(nets, sizes):
        ts = []
        for ls, kind, n in zip(labels, kinds, sz):
            if kind == "ct":
                ts.append(vecs[dims[ls[0]]].clone())
            else:
                ts.append(pool[at:at + n].clone().view([dims[l] for l in ls]))
            at += n
        out.append(ts)
    return out


# ------------------------------------------------------------- the library

_stream = None


def _side_stream():
    """The program's one stream for graph replays (a graph needs a stream
    other than the default one)."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def _create(tensors, labels, dims, case, path):
    net = htn.htn_create(tensors, labels, dims, [], compute=COMPUTE[case["dtype"]],
                         final_sum=FINAL[case.get("final", "plain")])
    if "lds" in case:
        htn.htn_set_option(net, htn.HTN_OPT_FUSED_LDS_BYTES, case["lds"])
        htn.htn_set_option(net, htn.HTN_OPT_FUSED_THREADS, case["threads"])
    if path is not None:
        htn.htn_set_path(net, path)
    return net


def _paths_of(case):
    """One path per network; None leaves the library's FLOP-greedy one."""
    if not case["samples"]:
        return [None] * len(_nets_of(case))
    return _paths(_key(case), case["samples"])


def _batch(nets, case, stream):
    out = htn.new_output(nets[0]).new_zeros(len(nets))
    b = htn.htn_batch_create(nets)
    if case.get("graph"):
        htn.htn_batch_set_graph(b, True)
    return {"batch": b, "out": out, "outs": htn.pointer_array([out[i:i + 1] for i in range(len(nets))]),
            "stream": stream}


def _circuit(case, seed):
    """The cut circuit; its rotation angles come from the seed."""
    if case["kind"] == "wires":
        return circuits.cut_wires(case["first"] + seed)
    return circuits.cut_marginal(case["first"] + seed, case["n_left"], case["n_right"], case["cuts"], case["layers"],
                                 case["kept"], case["kept"])


def _marginal_values(case, seed):
    """T1 [4]*c + [left], T2 [4]*c + [right]: every row a Dirichlet(1)
    quasi-distribution over its outputs."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = []
    for n in (case["left"], case["right"]):
        e = torch.empty(4 ** case["cuts"], n, dtype=torch.float64, device="cuda").exponential_(generator=gen)
        e /= e.sum(1, keepdim=True)
        out.append(e.to(TORCH[case["dtype"]]).view([4] * case["cuts"] + [n]))
    cw = torch.from_numpy(coeffs.CW.copy()).to("cuda", TORCH[case["dtype"]])
    return out + [cw.clone() for _ in range(case["cuts"])]


def _marginal_labels(c):
    return [list(range(c)) + [2 * c], list(range(c, 2 * c)) + [2 * c + 1]] + [[i, c + i] for i in range(c)]


def _uniforms(case, seed):
    """Per network one row of draws per gate cut."""
    rng = np.random.default_rng([2410, seed])
    return [[rng.random(case["draws"]) for k, ls in zip(kinds, labels) if k == "ct" and dims[ls[0]] == 6]
            for labels, dims, kinds in _nets_of(case)]


def _model_data(case, seed):
    """Rows of step features (log2 sizes / 8 and flags) and log durations."""
    rng = np.random.default_rng(seed)
    n = case["rows"]
    x = rng.uniform(0.0, 3.0, (n, htn.HTN_MODEL_FEATURES))
    x[:, 10:20] = rng.random((n, 10)) < 0.3
    t = 1.0 + 0.5 * x[:, 0] + 0.1 * rng.standard_normal(n)
    h, f = htn.HTN_MODEL_HIDDEN, htn.HTN_MODEL_FEATURES
    p = []
    for fan, k in ((f, h), (h, h), (h, 1)):
        p += [rng.uniform(-1, 1, k * fan) * math.sqrt(6.0 / fan), 0.1 * rng.standard_normal(k)]
    return x.astype(np.float32), t.astype(np.float32), np.concatenate(p).astype(np.float32)


def prepare(case, seed):
    fam = case["family"]
    if fam == "circuit":
        cn = _circuit(case, seed)
        ev = qteval.Evaluator([t for t in cn.tensors if hasattr(t, "instances")])
        entries = torch.zeros(ev.n_entries, dtype=torch.float64, device="cuda")
        qts = iter([entries[o:o + math.prod(s)].view(s) for o, s in zip(ev.entry_off, ev.shapes)])
        ts = [next(qts) if hasattr(t, "instances") else torch.from_numpy(np.array(t)).cuda() for t in cn.tensors]
        net = htn.htn_create(ts, cn.labels, cn.dims, cn.out_labels)
        return {"family": fam, "ev": ev, "entries": entries, "net": net, "out": htn.new_output(net)}
    if fam == "single":
        labels, dims, _ = _nets_of(case)[0]
        net = _create(_values(case, seed)[0], labels, dims, case, _paths_of(case)[0])
        return {"family": fam, "net": net, "out": htn.new_output(net)}
    if fam == "batch":
        nets = [_create(ts, labels, dims, case, path)
                for ts, (labels, dims, _), path in zip(_values(case, seed), _nets_of(case), _paths_of(case))]
        return {"family": fam, **_batch(nets, case, _side_stream() if case["graph"] else None)}
    if fam == "qpd":
        items, nets, src = [], [], _values(case, seed)
        for ts, (labels, dims, kinds), us, path in zip(src, _nets_of(case), _uniforms(case, seed), _paths_of(case)):
            gate = [i for i, k in enumerate(kinds) if k == "ct" and dims[labels[i][0]] == 6]
            s = htn_qpd.simplify(ts, labels, dims, [], gate, case["draws"], us, items)
            nets.append(_create(s.tensors, s.labels, s.dims, case, path))
        trunc = htn.htn_gather_create(items, COMPUTE[case["dtype"]]) if items else None
        return {"family": fam, "trunc": trunc, "src": src, **_batch(nets, case, None)}
    if fam == "marginal":
        c = case["cuts"]
        net = htn.htn_create(_marginal_values(case, seed), _marginal_labels(c),
                             [4] * (2 * c) + [case["left"], case["right"]], [2 * c, 2 * c + 1],
                             compute=COMPUTE[case["dtype"]], final_sum=FINAL[case["final"]])
        return {"family": fam, "net": net, "out": htn.new_output(net)}
    x, t, p = _model_data(case, seed)
    m = htn.htn_model_create(0)
    htn.htn_model_set_params(m, p)
    return {"family": fam, "model": m, "x": torch.from_numpy(x).cuda(), "t": torch.from_numpy(t).cuda(),
            "y": torch.zeros(case["rows"], device="cuda"), "grad": torch.zeros(p.size, device="cuda"),
            "loss": torch.zeros(1, device="cuda")}


def run(state):
    fam = state["family"]
    if fam == "circuit":
        htn.htn_qt_eval_run(state["ev"].handle, state["entries"])
        htn.htn_contract(state["net"], state["out"])
        return {"entries": state["entries"], "out": state["out"]}
    if fam in ("single", "marginal"):
        htn.htn_contract(state["net"], state["out"])
        return state["out"]
    if fam == "qpd" and state["trunc"] is not None:
        htn.htn_truncate_run(state["trunc"])
    if fam in ("batch", "qpd"):
        htn.htn_batch_run(state["batch"], state["outs"], state["stream"])
        return state["out"]
    htn.htn_model_forward(state["model"], state["x"], state["y"])
    htn.htn_model_gradients(state["model"], state["x"], state["t"], state["grad"], state["loss"])
    return {"y": state["y"], "grad": state["grad"], "loss": state["loss"]}


# ------------------------------------------------- work and 64-bit results

@functools.lru_cache(maxsize=8192)
def _order(sets, dims):
    """(order, multiplications) of a connected network whose every label
    joins two QTs: repeatedly the joined pair with the cheapest product."""
    live = {i: frozenset(s) for i, s in enumerate(sets)}
    at = {}
    for i, s in live.items():
        for l in s:
            at.setdefault(l, set()).add(i)

    def cost(i, j):
        return math.prod(dims[l] for l in live[i] | live[j])

    pairs = {tuple(sorted(p)): 0 for p in at.values() if len(p) == 2}
    pairs = {p: cost(*p) for p in pairs}
    order, mults, nxt = [], 0, len(sets)
    while pairs:
        (i, j), c = min(pairs.items(), key=lambda kv: (kv[1], kv[0]))
        mults += c
        summed = live[i] & live[j]
        order.append((i, j, summed))
        live[nxt] = (live.pop(i) | live.pop(j)) - summed
        pairs = {p: v for p, v in pairs.items() if i not in p and j not in p}
        for l in live[nxt]:
            at[l] = (at[l] - {i, j}) | {nxt}
            p = tuple(sorted(at[l]))
            if p not in pairs:
                pairs[p] = cost(*p)
        nxt += 1
    return order, mults


def _qt_sets(labels, kinds):
    return tuple(tuple(ls) for ls, k in zip(labels, kinds) if k == "qt")


def work(case):
    fam = case["family"]
    if fam == "circuit":
        cn = _circuit(case, 0)
        flops, nbytes = 0, 0
        for t in cn.tensors:
            if hasattr(t, "instances"):
                # 14 flops per amplitude of a one-qubit unitary, 6 per
                # amplitude of the measurement
                flops += sum((sum(14 if o[0] == "u" else 1 for o in i.ops) + 6) << i.n_qubits for i in t.instances)
                nbytes += sum(96 * len(i.ops) + 32 * i.n_qubits for i in t.instances) + 8 * math.prod(t.shape)
        out = math.prod(cn.dims[l] for l in cn.out_labels)
        flops += 2 * out * 4 ** case.get("cuts", 2)
        return {"bytes": nbytes + 8 * out, "flops": flops}
    if fam in ("single", "batch", "qpd"):
        b = BYTES[case["dtype"]]
        nbytes = flops = 0
        if fam == "qpd":
            kept = [[len(np.unique(np.minimum((u * 6).astype(int), 5))) for u in us] for us in _uniforms(case, 0)]
        for i, (labels, dims, kinds) in enumerate(_nets_of(case)):
            dims = list(dims)
            if fam == "qpd":
                it = iter(kept[i])
                gate = [ls[0] for k, ls in zip(kinds, labels) if k == "ct" and dims[ls[0]] == 6]
                for l in gate:
                    dims[l] = next(it)
            nbytes += b * sum(math.prod(dims[l] for l in ls) for ls in labels) + 8
            flops += 2 * _order(_qt_sets(labels, kinds), tuple(dims))[1]
        return {"bytes": nbytes, "flops": flops}
    if fam == "marginal":
        k, m, n = 4 ** case["cuts"], case["left"], case["right"]
        b = BYTES[case["dtype"]]
        return {"bytes": b * (k * (m + n) + 16 * case["cuts"]) + 8 * m * n,
                "flops": 2 * m * n * k + 2 * 4 * case["cuts"] * k * min(m, n)}
    f, h, r = htn.HTN_MODEL_FEATURES, htn.HTN_MODEL_HIDDEN, case["rows"]
    w = f * h + h * h + h
    return {"bytes": 4 * (2 * r * (f + 1) + r + 2 * (w + 2 * h + 1)), "flops": 2 * r * (w + w + 2 * w - f * h)}


def _contract64(tensors, sets, dims):
    order, _ = _order(sets, tuple(dims))
    live = {i: (t, list(s)) for i, (t, s) in enumerate(zip(tensors, sets))}
    nxt = len(sets)
    for i, j, summed in order:
        (a, la), (b, lb) = live.pop(i), live.pop(j)
        s = sorted(summed)
        t = torch.tensordot(a, b, dims=([la.index(l) for l in s], [lb.index(l) for l in s]))
        live[nxt] = (t, [l for l in la if l not in summed] + [l for l in lb if l not in summed])
        nxt += 1
    return live[nxt - 1][0].reshape(())


def _exact_nets(case, values, draws=None):
    """Every network's value in FP64: each cut's weights scale one of the two
    QTs that carry its label, then pairwise products."""
    res = []
    for n, (ts, (labels, dims, kinds)) in enumerate(zip(values, _nets_of(case))):
        dims = list(dims)
        weight, kept = {}, {}
        gates = 0
        for t, ls, k in zip(ts, labels, kinds):
            if k != "ct":
                continue
            w = t.double()
            if draws is not None and dims[ls[0]] == 6:
                u = draws[n][gates]
                gates += 1
                c = w.cpu().numpy()
                gamma = np.abs(c).sum()
                idx = np.searchsorted(np.cumsum(np.abs(c)) / gamma, u, side="right")
                cnt = np.bincount(np.minimum(idx, len(c) - 1), minlength=len(c))
                w = torch.from_numpy(cnt * gamma * np.sign(c) / len(u)).to(t.device)
                kept[ls[0]] = torch.from_numpy(np.nonzero(cnt)[0]).to(t.device)
                w = w[kept[ls[0]]]
                dims[ls[0]] = len(w)
            weight[ls[0]] = w
        qts, sets = [], []
        done = set()
        for t, ls, k in zip(ts, labels, kinds):
            if k != "qt":
                continue
            t = t.double()
            for ax, l in enumerate(ls):
                if l in kept:
                    t = t.index_select(ax, kept[l])
                if l not in done:
                    done.add(l)
                    t = t * weight[l].view([-1 if a == ax else 1 for a in range(t.dim())])
            qts.append(t)
            sets.append(tuple(ls))
        res.append(_contract64(qts, tuple(sets), dims))
    return torch.stack(res)


def _apply(psi, op, n):
    """One op on a batch of states [..., 2 x n qubits] (complex128)."""
    off = psi.dim() - n
    if op[0] == "u":
        u = torch.from_numpy(np.array(op[2], dtype=np.complex128)).to(psi.device)
        return torch.movedim(torch.tensordot(u, psi, dims=([1], [off + op[1]])), 0, off + op[1])
    psi = psi.clone()
    view = torch.movedim(psi, (off + op[1], off + op[2]), (0, 1))
    view[1, 1] *= -1.0  # cz
    return psi


PAULI = {"I": np.eye(2), "X": circuits.X, "Y": circuits.Y, "Z": circuits.Z}


def _instance64(inst, states):
    """An instance's outputs; evolved states are kept by their preparation
    and gates, which instances of several observables share."""
    n = inst.n_qubits
    key = (tuple(np.asarray(v).tobytes() for v in inst.init), id(inst.ops[0][2]), len(inst.ops))
    if key not in states:
        psi = torch.ones((), dtype=torch.complex128, device="cuda")
        for v in inst.init:
            psi = torch.tensordot(psi, torch.from_numpy(np.array(v, dtype=np.complex128)).cuda(), dims=0)
        for op in inst.ops:
            psi = _apply(psi, op, n)
        states[key] = psi
    psi = states[key]
    phi = psi
    for q, p in enumerate(inst.observable):
        if p != "I":
            phi = _apply(phi, ("u", q, PAULI[p]), n)
    prob = (psi.conj() * phi).real
    rest = [q for q in range(n) if q not in inst.kept]
    prob = prob.permute(list(inst.kept) + rest).reshape(1 << len(inst.kept), -1)
    return prob.sum(1).cpu().numpy()


def _exact_circuit(case, seed):
    cn = _circuit(case, seed)
    entries, tensors = [], []
    for t in cn.tensors:
        if not hasattr(t, "instances"):
            tensors.append(np.asarray(t, dtype=np.float64))
            continue
        states = {}
        outs = [_instance64(i, states) for i in t.instances]
        e = np.array([sum(c * outs[k][x] for k, x, c in terms) for terms in t.terms])
        entries.append(e)
        tensors.append(e.reshape(t.shape))
    args = []
    for t, ls in zip(tensors, cn.labels):
        args += [t, ls]
    out = np.einsum(*args, list(cn.out_labels), optimize=True)
    return {"entries": np.concatenate(entries), "out": np.asarray(out, dtype=np.float64).reshape(-1)}


def _exact_model(case, seed):
    x, t, p = (torch.from_numpy(a.astype(np.float64)) for a in _model_data(case, seed))
    f, h = htn.HTN_MODEL_FEATURES, htn.HTN_MODEL_HIDDEN
    p.requires_grad_(True)
    w1, b1, w2, b2, w3, b3 = torch.split(p, [h * f, h, h * h, h, h, 1])
    a = torch.relu(x @ w1.view(h, f).T + b1)
    a = torch.relu(a @ w2.view(h, h).T + b2)
    y = a @ w3 + b3
    loss = ((y - t) ** 2).mean()
    (g,) = torch.autograd.grad(loss, p)
    return {"y": y.detach(), "grad": g, "loss": loss.detach().reshape(1)}


def exact(case, seed):
    fam = case["family"]
    if fam == "circuit":
        return _exact_circuit(case, seed)
    if fam == "single":
        return _exact_nets(case, _values(case, seed)).reshape(1)
    if fam == "batch":
        return _exact_nets(case, _values(case, seed))
    if fam == "qpd":
        return _exact_nets(case, _values(case, seed), _uniforms(case, seed))
    if fam == "marginal":
        ts = [t.double() for t in _marginal_values(case, seed)]
        fold = ts[0]
        for cw in ts[2:]:  # label i of T1 becomes label c + i
            fold = torch.tensordot(fold, cw, dims=([0], [0]))
        # axes now: [left, c, c + 1, ...]
        return (fold.reshape(case["left"], -1) @ ts[1].reshape(-1, case["right"])).reshape(-1)
    return _exact_model(case, seed)
