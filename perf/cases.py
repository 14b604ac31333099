"""Performance cases: the work that programs have this library do.

A case is a dict of plain values; `listed()` holds the fixed ones, `draw(rng)`
gives further ones of the same ranges.  `prepare(case, seed)` builds what a
program has in hand before the call (plan, workspace, device leaves),
`run(state)` is one pass through the public entry points, `work(case)` the
bytes and operations the pass cannot do without, and `exact(case, seed)` the
same outputs from plain torch complex128 tensor algebra.

Kinds of case:
  circuit  amplitudes of a random grid circuit (open qubits = output axes),
           unsliced (Plan.contract) or over slice ids (Plan.contract_sliced)
  rrg      random 3-regular graph of rank-3 Gaussian tensors, all slices
  random   random network with hyperedges, open indices and dimensions 2 / 4
  qaoa     every term of a MAX-CUT QAOA energy in one batch (Batch.contract)
  grad     amplitudes and the gradients of all two-qubit gate tensors
           (Plan.contract_sliced + Plan.backward, or the autograd wrapper)
  node     one pairwise contraction, classes of 2^h, 2^m, 2^n, 2^k values
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

from tn_inputs import configs, qaoa
from tn_inputs.circuits import circuit_network, gate_leaves
from tn_inputs.graphs import random_network, rrg_network
from tn_inputs.greedy import find_tree, width_cost
from tn_inputs.network import Network, Tree


def listed():
    return [
        # one amplitude of a small circuit in double precision: the smallest
        # call, where a program loops over bitstrings and latency counts
        dict(name="amp_3x3x8_c128", kind="circuit", R=3, C=3, m=8, open=0, width=0, slices=0, inflight=0,
             decompose="none", precision="c128"),
        # a training loop on a small circuit through the autograd wrapper
        dict(name="train_4x4x8", kind="grad", R=4, C=4, m=8, open=2, precision="c64_4m", autograd=True),
        # the random-tensor benchmark network of the repository (120 vertices,
        # width 20): a cancelling sum, contracted in double precision
        dict(name="rrg_120_c128", kind="rrg", n=120, graph=0, width=20, precision="c128"),
        # a QAOA energy: 81 light-cone networks of up to 200 leaves
        dict(name="qaoa_54_3", kind="qaoa", n=54, p=3, precision="c64_4m"),
        # gradients of a mid-sized circuit: large intermediates, recomputation
        dict(name="grad_5x6x10", kind="grad", R=5, C=6, m=10, open=3, precision="c64_4m", autograd=False),
        # correlated amplitudes in double precision, unsliced
        dict(name="amps_5x5x12_c128", kind="circuit", R=5, C=5, m=12, open=3, width=0, slices=0, inflight=0,
             decompose="none", precision="c128"),
        # the 54-qubit circuit of the benchmark with small slices, several in
        # flight: the ordinary large job (one of its many calls)
        dict(name="slices_6x9x12", kind="circuit", R=6, C=9, m=12, open=6, width=26, slices=4, inflight=2,
             decompose="none", precision="c64_4m"),
        # one slice of the hyperedge variant at the benchmark's full width
        dict(name="slice_6x9x12_hyper", kind="circuit", R=6, C=9, m=12, open=6, width=30, slices=1, inflight=1,
             decompose="swap_diag", precision="c64_4m"),
        # single contractions: matrix-core shapes in the other two complex64
        # modes, a write-bound one and a long reduction to few outputs
        dict(name="node_bf16x3", kind="node", h=1, m=11, n=12, k=13, shuffled=False, precision="c64_bf16x3"),
        dict(name="node_3m", kind="node", h=0, m=12, n=12, k=12, shuffled=False, precision="c64_3m"),
        dict(name="node_fewsum", kind="node", h=0, m=13, n=13, k=2, shuffled=False, precision="c64_4m"),
        dict(name="node_reduce", kind="node", h=0, m=3, n=2, k=22, shuffled=True, precision="c64_4m"),
    ]


# Most complex multiply-adds (log2) of a drawn case: below the largest listed one.
_MAX_MACS = {"c64_4m": 40.0, "c64_3m": 40.0, "c64_bf16x3": 40.0, "c128": 37.0}


def draw(rng):
    kind = rng.choice(["circuit", "circuit", "circuit", "rrg", "random", "qaoa", "grad", "grad", "node", "node", "node"])
    prec = rng.choice(["c64_4m", "c64_4m", "c64_4m", "c64_3m", "c64_bf16x3", "c128", "c128"])
    if kind == "circuit":
        while True:
            R = rng.randint(3, 6)
            C = rng.randint(R, min(9, R + 3))
            c = dict(kind="circuit", R=R, C=C, m=rng.randint(4, 14), open=rng.randint(3, 6),
                     width=0, slices=0, inflight=0, decompose=rng.choice(["none", "none", "swap_diag"]),
                     precision=prec)
            if rng.random() < 0.5:
                c.update(width=rng.randint(16, 27), slices=rng.choice([1, 2, 3, 5, 8, 13]), inflight=rng.randint(1, 4))
            tree, _ = _tree(_key(c))
            # a width that the finder's greedy slicer can reach in few steps,
            # tensors of at most 2^28 values, and bounded work
            if c["width"] and tree.meta["W"] - c["width"] > 20:
                continue
            if tree.meta.get("W_s", tree.meta["W"]) <= 28 and math.log2(_macs(c)) <= _MAX_MACS[prec]:
                return c
    if kind == "rrg":
        return dict(kind="rrg", n=2 * rng.randint(15, 60), graph=rng.randint(0, 9), width=rng.randint(14, 20),
                    precision="c128")
    if kind == "random":
        return dict(kind="random", n_leaves=rng.randint(6, 24), max_rank=rng.randint(5, 7), n_out=rng.randint(3, 7),
                    graph=rng.randint(0, 99), precision=prec)
    if kind == "qaoa":
        return dict(kind="qaoa", n=2 * rng.randint(4, 27), p=rng.choice([1, 2, 2, 3]),
                    precision=rng.choice(["c64_4m", "c64_4m", "c128"]))
    if kind == "grad":
        while True:
            R = rng.randint(3, 5)
            c = dict(kind="grad", R=R, C=rng.randint(R, 6), m=rng.randint(4, 12), open=rng.randint(2, 4),
                     precision=prec, autograd=rng.random() < 0.4)
            tree, _ = _tree(_key(c))
            if tree.meta["W"] <= 26 and math.log2(_macs(c)) <= _MAX_MACS[prec]:
                return c
    while True:
        h, m, n = rng.choice([0, 0, 1, 2, 3]), rng.randint(0, 14), rng.randint(0, 14)
        k = rng.choice([rng.randint(0, 4), rng.randint(3, 13), rng.randint(8, 22)])
        if max(h + m + n, h + m + k, h + n + k) <= 26 and 12 <= h + m + n + k <= _MAX_MACS[prec] - 1:
            return dict(kind="node", h=h, m=m, n=n, k=k, shuffled=rng.random() < 0.5, precision=prec)


# ------------------------------------------------------------------ structures

def _key(case):
    """The fields that fix a case's network structure and tree."""
    return tuple(sorted((k, v) for k, v in case.items()
                        if k in ("kind", "R", "C", "m", "open", "width", "decompose", "n", "graph", "n_leaves",
                                 "max_rank", "n_out")))


def _open_qubits(R, C, count):
    """`count` qubits around the centre of the grid (two rows of three first)."""
    r, c = R // 2 - 1, C // 2 - 1
    block = [(r + i) * C + c + j for i in (0, 1) for j in (0, 1, 2) if c + j < C]
    rest = [q for q in range(R * C) if q not in block]
    return tuple(sorted((block + rest)[:count]))


def _network(key, seed):
    """The network of a structure with the tensors of `seed`."""
    c = dict(key)
    rng = np.random.default_rng(seed)
    if c["kind"] in ("circuit", "grad"):
        N = c["R"] * c["C"]
        bits = int(rng.integers(0, 2 ** N, dtype=np.uint64))
        return circuit_network(c["R"], c["C"], c["m"], seed, bits, open_qubits=_open_qubits(c["R"], c["C"], c["open"]),
                               decompose=c.get("decompose", "none"))
    if c["kind"] == "rrg":
        net = rrg_network(c["n"], 3, seed=c["graph"])
        scale = 2.0 ** -0.75 * math.sqrt(0.5)
    else:
        net = random_network(c["n_leaves"], 7 * c["n_leaves"] // 5, c["max_rank"], c["graph"], n_out=c["n_out"], dims=(2, 4),
                             hyper=True)
        scale = 1.0
    return net.with_leaves([scale * (rng.normal(size=t.shape) + 1j * rng.normal(size=t.shape)) for t in net.leaves])


@functools.lru_cache(maxsize=None)
def _tree(key):
    """(tree, sliced indices) of a structure: the repository's cached tree of
    its benchmark networks, the best of four seeded greedy trees otherwise."""
    c = dict(key)
    if c["kind"] == "rrg" and c["n"] == 120 and c["width"] == 20:
        _, tree, sliced = configs.load("cfg2", c["graph"])
        return tree, sliced
    if c["kind"] == "circuit" and (c["R"], c["C"], c["m"], c["open"], c["width"], c["decompose"]) == \
            (6, 9, 12, 6, 30, "swap_diag"):
        _, tree, sliced = configs.load("cfg5h")
        return tree, sliced
    net = _network(key, 0)
    if c["kind"] == "random":
        tree = find_tree(net, seed=0, trials=1)
    else:
        tree = find_tree(net, seed=0, trials=4, slice_width=c.get("width") or None)
    return tree, list(tree.meta.get("sliced", []))


@functools.lru_cache(maxsize=None)
def _cost(key):
    """Complex multiply-adds of one slice."""
    tree, sliced = _tree(key)
    mask = 0
    for e in sliced:
        mask |= 1 << e
    return 2.0 ** width_cost(_network(key, 0), tree, mask)[1]


@functools.lru_cache(maxsize=None)
def _terms(n, p):
    """Edges and trees of a QAOA instance's terms (structure only)."""
    edges, gammas, betas = qaoa.instance(n, p, 0)
    nets = [qaoa.term_network(edges, gammas, betas, j, k) for j, k in edges]
    return edges, [find_tree(net, seed=0, trials=4) for net in nets], nets


def _term_networks(case, seed):
    edges, trees, _ = _terms(case["n"], case["p"])
    rng = np.random.default_rng(seed)
    gammas, betas = rng.uniform(0.0, np.pi, case["p"]), rng.uniform(0.0, np.pi, case["p"])
    return [qaoa.term_network(edges, gammas, betas, j, k) for j, k in edges], trees


def _node_network(case):
    """Two leaves A(H, M, K) and B(H, N, K) with outputs (H, M, N), one binary
    index per bit: in that axis order, or in a shuffled one."""
    ids, start = {}, 0
    for name in "hmnk":
        ids[name] = list(range(start, start + case[name]))
        start += case[name]
    a, b, o = ids["h"] + ids["m"] + ids["k"], ids["h"] + ids["n"] + ids["k"], ids["h"] + ids["m"] + ids["n"]
    if case["shuffled"]:
        rng = np.random.default_rng(case["h"] + 16 * case["m"] + 256 * case["n"] + 4096 * case["k"])
        a, b, o = ([x[i] for i in rng.permutation(len(x))] for x in (a, b, o))
    return Network([], [a, b], [2] * start, o), Tree(np.array([0], np.int32), np.array([1], np.int32))


def _node_leaves(case, net, seed):
    """Gaussian operands, complex64 values (complex128 for c128 plans)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.complex128 if case["precision"] == "c128" else torch.complex64
    return [torch.randn((2,) * len(ix), dtype=dt, device="cuda", generator=g) for ix in net.leaf_idx]


def _slice_ids(case, sliced, dims, seed):
    d = math.prod(dims[e] for e in sliced)
    n = min(d, case.get("slices") or d)
    return None if n == d else sorted(int(x) for x in np.random.default_rng(seed + 1).choice(d, n, replace=False))


def _macs(case):
    """Complex multiply-adds of one forward pass."""
    if case["kind"] == "node":
        return 2.0 ** (case["h"] + case["m"] + case["n"] + case["k"])
    if case["kind"] == "qaoa":
        _, trees, nets = _terms(case["n"], case["p"])
        return sum(2.0 ** width_cost(net, tree)[1] for net, tree in zip(nets, trees))
    key = _key(case)
    d = 2.0 ** len(_tree(key)[1])
    return _cost(key) * min(d, case.get("slices") or d)


# ------------------------------------------------------------------ the cases

def _device(arrays, precision):
    dt = torch.complex128 if precision == "c128" else torch.complex64
    return [torch.from_numpy(np.ascontiguousarray(t)).to(device="cuda", dtype=dt) for t in arrays]


def prepare(case, seed):
    from paper_2002_01935_amd.binding import Batch, Plan
    kind, prec = case["kind"], case["precision"]
    if kind == "qaoa":
        nets, trees = _term_networks(case, seed)
        plans = [Plan(net, tree, precision=prec) for net, tree in zip(nets, trees)]
        batch = Batch(plans)
        ws = batch.workspace()
        batch.prepare(ws)
        energy_terms = torch.empty(len(plans), dtype=plans[0].storage_dtype, device="cuda")
        return dict(kind=kind, batch=batch, ws=ws, leaves=[_device(net.leaves, prec) for net in nets],
                    terms=energy_terms, outs=[energy_terms[i] for i in range(len(plans))])
    if kind == "node":
        net, tree = _node_network(case)
        plan = Plan(net, tree, precision=prec)
        return dict(kind="contract", plan=plan, leaves=_node_leaves(case, net, seed), ws=plan.workspace(),
                    out=torch.empty(plan.out_shape, dtype=plan.storage_dtype, device="cuda"))
    key = _key(case)
    net, (tree, sliced) = _network(key, seed), _tree(key)
    plan = Plan(net, tree, sliced=sliced, precision=prec, max_inflight_slices=case.get("inflight", 0))
    leaves = _device(net.leaves, prec)
    if kind == "grad":
        wrt = gate_leaves(net)
        if case["autograd"]:
            for v in wrt:
                leaves[v].requires_grad_(True)
            return dict(kind="autograd", plan=plan, leaves=leaves, wrt=wrt)
        size = [leaves[v].numel() for v in wrt]
        flat = torch.empty(sum(size), dtype=plan.storage_dtype, device="cuda")
        grads = [g.reshape(leaves[v].shape) for v, g in zip(wrt, flat.split(size))]
        ws = plan.workspace(plan.backward_info(wrt)["workspace_bytes"])
        return dict(kind="grad", plan=plan, leaves=leaves, wrt=wrt, ws=ws, flat=flat, grads=grads,
                    out=torch.empty(plan.out_shape, dtype=torch.complex128, device="cuda"))
    ws = plan.workspace()
    if not sliced:
        return dict(kind="contract", plan=plan, leaves=leaves, ws=ws,
                    out=torch.empty(plan.out_shape, dtype=plan.storage_dtype, device="cuda"))
    return dict(kind="sliced", plan=plan, leaves=leaves, ws=ws, ids=_slice_ids(case, sliced, net.idx_dim, seed),
                out=torch.empty(plan.out_shape, dtype=torch.complex128, device="cuda"))


def run(s):
    if s["kind"] == "contract":
        return s["plan"].contract(s["leaves"], out=s["out"], workspace=s["ws"])
    if s["kind"] == "sliced":
        return s["plan"].contract_sliced(s["leaves"], slice_ids=s["ids"], out=s["out"], workspace=s["ws"])
    if s["kind"] == "qaoa":
        s["batch"].contract(s["leaves"], s["ws"], outs=s["outs"])
        return s["terms"]
    if s["kind"] == "grad":
        # L = sum |amplitude|^2: dL/d(amplitude) = 2 amplitude
        out = s["plan"].contract_sliced(s["leaves"], out=s["out"], workspace=s["ws"])
        s["plan"].backward(s["leaves"], 2.0 * out, s["wrt"], grads=s["grads"], workspace=s["ws"])
        return [out, s["flat"]]
    from paper_2002_01935_amd.autograd import contract
    for v in s["wrt"]:
        s["leaves"][v].grad = None
    out = contract(s["plan"], s["leaves"])
    out.abs().square().sum().backward()
    return [out.detach(), torch.cat([s["leaves"][v].grad.reshape(-1) for v in s["wrt"]])]


def work(case):
    eb = 16 if case["precision"] == "c128" else 8
    macs = _macs(case)
    if case["kind"] == "node":
        h, m, n, k = (case[x] for x in "hmnk")
        return dict(bytes=eb * (2.0 ** (h + m + k) + 2.0 ** (h + n + k) + 2.0 ** (h + m + n)), flops=8.0 * macs)
    if case["kind"] == "qaoa":
        nets = _terms(case["n"], case["p"])[2]
        return dict(bytes=eb * float(sum(sum(t.size for t in net.leaves) + 1 for net in nets)), flops=8.0 * macs)
    net = _network(_key(case), 0)
    n_in, n_out = sum(t.size for t in net.leaves), math.prod(net.idx_dim[e] for e in net.out_idx)
    if case["kind"] == "grad":
        # the forward pass, and two products per node on the way back
        n_grad = sum(net.leaves[v].size for v in gate_leaves(net))
        return dict(bytes=float(eb * (n_in + n_grad) + 16 * n_out), flops=24.0 * macs)
    return dict(bytes=float(eb * n_in + 16 * n_out), flops=8.0 * macs)


# ------------------------------------------------------------------ values in 64 bits

def _permuted(x, ids, target, dims):
    """Flat copy of x (row-major over `ids`) in the axis order `target`."""
    if list(ids) == list(target):
        return x
    stride, s = {}, 1
    for e in reversed(ids):
        stride[e] = s
        s *= dims[e]
    runs = []                       # target axes, last first, merged where they stay adjacent: (size, stride in x)
    for e in reversed(target):
        if runs and runs[-1][0] * runs[-1][1] == stride[e]:
            runs[-1] = (runs[-1][0] * dims[e], runs[-1][1])
        else:
            runs.append((dims[e], stride[e]))
    out = torch.empty_like(x)
    step = 1 << 26
    for at in range(0, x.numel(), step):
        i = torch.arange(at, min(at + step, x.numel()), device=x.device)
        src = torch.zeros_like(i)
        for size, st in runs:
            src += (i % size) * st
            i //= size
        out[at:at + step] = x[src]
    return out


def _product(a, ia, b, ib, target, dims):
    """Sum over the indices outside `target` of a * b, as a flat tensor."""
    sa, sb, st = set(ia), set(ib), set(target)
    H = [e for e in target if e in sa and e in sb]
    M = [e for e in target if e in sa and e not in sb]
    N = [e for e in target if e not in sa]
    K = [e for e in ia if e not in st and e in sb]
    a, ia = _summed(a, ia, [e for e in ia if e not in st and e not in sb], dims)
    b, ib = _summed(b, ib, [e for e in ib if e not in st and e not in sa], dims)
    h, m, n, k = (math.prod(dims[e] for e in x) for x in (H, M, N, K))
    a = _permuted(a, ia, H + M + K, dims).reshape(h, m, k)
    b = _permuted(b, ib, H + K + N, dims).reshape(h, k, n)
    c = a @ b if k > 1 else a * b
    return _permuted(c.reshape(-1), H + M + N, target, dims)


def _summed(x, ids, gone, dims):
    if not gone:
        return x, ids
    left = [e for e in ids if e not in set(gone)]
    return _permuted(x, ids, left + list(gone), dims).reshape(-1, math.prod(dims[e] for e in gone)).sum(1), left


def _kept(net, tree):
    """Indices of every node: those below it that an output or a leaf outside holds."""
    n = net.n_leaves
    total, below, kept = {}, [], []
    for ix in net.leaf_idx:
        for e in ix:
            total[e] = total.get(e, 0) + 1
        below.append({e: 1 for e in ix})
        kept.append(list(ix))
    for l, r in zip(tree.left, tree.right):
        cnt = dict(below[l])
        for e, c in below[r].items():
            cnt[e] = cnt.get(e, 0) + c
        cnt = {e: c for e, c in cnt.items() if e in net.out_idx or c < total[e]}
        below.append(cnt)
        kept.append(list(cnt))
    if len(kept) > n:
        kept[-1] = list(net.out_idx)
    return kept


def _contract(net, tree, values, fixed, keep=False):
    """The network's value with the indices of `fixed` at the given values;
    with `keep`, the values of all nodes instead."""
    n, dims = net.n_leaves, net.idx_dim
    kept = [[e for e in ids if e not in fixed] for ids in _kept(net, tree)]
    val = []
    for ids, t in zip(net.leaf_idx, values):
        val.append(t.reshape([dims[e] for e in ids])[tuple(fixed.get(e, slice(None)) for e in ids)].reshape(-1))
    for k, (l, r) in enumerate(zip(tree.left, tree.right)):
        val.append(_product(val[l], kept[l], val[r], kept[r], kept[n + k], dims))
        if not keep:
            val[l] = val[r] = None
    return (val, kept) if keep else val[-1]


def _rounded(leaves, precision):
    """The leaves as the plan receives them, promoted to complex128 (exact)."""
    return [t.to(torch.complex128) for t in _device(leaves, precision)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "qaoa":
        nets, trees = _term_networks(case, seed)
        return torch.stack([_contract(net, tree, _rounded(net.leaves, case["precision"]), {})[0]
                            for net, tree in zip(nets, trees)])
    if kind == "node":
        net, tree = _node_network(case)
        values = [t.to(torch.complex128).reshape(-1) for t in _node_leaves(case, net, seed)]
        return _contract(net, tree, values, {}).reshape((2,) * len(net.out_idx))
    key = _key(case)
    net, (tree, sliced) = _network(key, seed), _tree(key)
    values, dims = _rounded(net.leaves, case["precision"]), net.idx_dim
    shape = [dims[e] for e in net.out_idx]
    if kind == "grad":
        val, kept = _contract(net, tree, values, {}, keep=True)
        grad = {len(val) - 1: 2.0 * val[-1]}
        n = net.n_leaves
        for k in range(len(tree.left) - 1, -1, -1):
            l, r, g = int(tree.left[k]), int(tree.right[k]), grad.pop(n + k)
            grad[l] = _product(g, kept[n + k], val[r].conj().resolve_conj(), kept[r], kept[l], dims)
            grad[r] = _product(g, kept[n + k], val[l].conj().resolve_conj(), kept[l], kept[r], dims)
        return [val[-1].reshape(shape), torch.cat([grad[v] for v in gate_leaves(net)])]
    ids = _slice_ids(case, sliced, dims, seed) if sliced else [0]
    total = 0
    for sid in range(math.prod(dims[e] for e in sliced)) if ids is None else ids:
        fixed = {}
        for e in reversed(sliced):          # first sliced index most significant
            fixed[e] = sid % dims[e]
            sid //= dims[e]
        total = total + _contract(net, tree, values, fixed)
    return total.reshape(shape)
