"""Groups of small contractions run by one workgroup (tiny_tree_kernel)
against the oracle: networks with sliced and strided leaves, hyperedges and
dimensions 2 and 4, contractions around the largest size a group takes, a
chain longer than one group holds (cut into several), several slices in
flight, forward and reverse."""

import numpy as np
import pytest

from tests.gpu_util import TOL_C64, TOL_C128, c64_leaves, note, rel, to_dev
from tn_inputs.graphs import random_network
from tn_inputs.greedy import find_tree
from tn_inputs.network import Network, Tree

pytestmark = pytest.mark.gpu


def _chain(length, rng):
    """A 4-vector, length - 1 unitary 4 x 4 matrices with shuffled axes, open at the end."""
    leaves, idx = [rng.normal(size=4) + 1j * rng.normal(size=4)], [[0]]
    for v in range(1, length):
        q = np.linalg.qr(rng.normal(size=(4, 4)) + 1j * rng.normal(size=(4, 4)))[0]
        flip = bool(rng.integers(2))
        leaves.append(np.ascontiguousarray(q.T if flip else q))
        idx.append([v, v - 1] if flip else [v - 1, v])
    net = Network(leaves, idx, [4] * length, [length - 1])
    left, right, node = [], [], 0
    for v in range(1, length):
        left.append(node)
        right.append(v)
        node = length + v - 1
    return net, Tree(np.array(left, np.int32), np.array(right, np.int32)), []


def _pair_tail(out_bits, k_bits, rng):
    """(A, B) with 2^out_bits outputs and 2^k_bits summed values, then a vector
    on one of the outputs: two contractions, the first one of the given size."""
    m = (out_bits + 1) // 2
    M, N, K = list(range(m)), list(range(m, out_bits)), list(range(out_bits, out_bits + k_bits))
    idx = [list(rng.permutation(M + K)), list(rng.permutation(N + K)), [M[0]]]
    idx = [[int(e) for e in ix] for ix in idx]
    leaves = [rng.normal(size=(2,) * len(ix)) + 1j * rng.normal(size=(2,) * len(ix)) for ix in idx]
    out = [int(e) for e in rng.permutation(M[1:] + N)]
    return Network(leaves, idx, [2] * (out_bits + k_bits), out), Tree(np.array([0, 3], np.int32), np.array([1, 2], np.int32)), []


def _random(seed):
    net = random_network(12, 18, 5, seed=500 + seed, n_out=2, dims=(2, 4), hyper=True)
    return net, find_tree(net, seed=seed, trials=2), [e for e in range(net.n_idx) if e not in net.out_idx][:3]


CASES = {"chain-40": lambda r: _chain(40, r), "chain-700": lambda r: _chain(700, r)}
CASES.update({f"pair-{o}-{k}": lambda r, o=o, k=k: _pair_tail(o, k, r)
              for o, k in ((2, 0), (2, 8), (6, 6), (10, 2), (10, 3), (11, 1), (9, 3), (4, 7))})
CASES.update({f"random-{s}": lambda r, s=s: _random(s) for s in range(3)})


@pytest.mark.parametrize("prec", ["c64_4m", "c128"])
@pytest.mark.parametrize("name", CASES)
def test_small_groups(oracle_lib, name, prec):
    import torch

    from paper_2002_01935_amd.binding import Plan
    rng = np.random.default_rng(sum(map(ord, name)))
    net, tree, sliced = CASES[name](rng)
    net.check()
    tol = TOL_C128 if prec == "c128" else TOL_C64
    ref_net = net if prec == "c128" else c64_leaves(net)
    plan = Plan(net, tree, sliced=sliced, precision=prec, max_inflight_slices=3)
    d = plan.info()["d_sliced"]
    ids = [s for s in range(d) if s % 4 != 2]
    leaves = to_dev(net, prec)
    ref = oracle_lib.contract(ref_net, tree, sliced=sliced, slice_ids=ids)
    got = plan.contract_sliced(leaves, slice_ids=ids)
    wrt = list(range(0, net.n_leaves, 1 + net.n_leaves // 50))
    shape = tuple(net.idx_dim[e] for e in net.out_idx)
    go = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    grads = plan.backward(leaves, torch.from_numpy(go), wrt, slice_ids=ids)
    torch.cuda.synchronize()
    e = rel(got.cpu().numpy(), ref)
    if not sliced:
        e = max(e, rel(plan.contract(leaves).cpu().numpy(), ref))
    refs = oracle_lib.grad(ref_net, tree, go, wrt, sliced=sliced, slice_ids=ids)
    eg = max(rel(g.cpu().numpy(), r) for g, r in zip(grads, refs))
    note("small groups", name, prec, "%.2e, gradients %.2e" % (e, eg), {n["kernel"] for n in plan.nodes()})
    assert e < tol and eg < tol
    if name.startswith(("chain", "random")) or name in ("pair-2-0", "pair-10-2", "pair-9-3"):
        assert any(n["kernel"] == "tiny_tree_kernel" for n in plan.nodes()), name
    if name in ("pair-10-3", "pair-11-1"):
        assert plan.nodes()[0]["kernel"] != "tiny_tree_kernel", name


@pytest.mark.parametrize("prec", ["c64_4m", "c128"])
def test_batch_levels(oracle_lib, prec):
    """A batch whose networks need several stages of groups (a chain longer
    than one group), and contractions of every way the batch's level kernel
    shares a sum: one thread, one wavefront or one workgroup per output."""
    import torch

    from paper_2002_01935_amd.binding import Batch, Plan
    rng = np.random.default_rng(7)
    nets = [_chain(400, rng)] + [_pair_tail(o, k, rng) for o, k in ((13, 0), (14, 2), (10, 5), (12, 6), (13, 8), (14, 7),
                                                                    (2, 9), (8, 12), (4, 15), (9, 12), (1, 6))]
    nets += [_chain(200, rng)] + [_random(s)[:2] + ([],) for s in range(3)]
    plans = [Plan(net, tree, precision=prec) for net, tree, _ in nets]
    batch = Batch(plans)
    ws = batch.workspace()
    batch.prepare(ws)
    leaves = [to_dev(net, prec) for net, _, _ in nets]
    tol = TOL_C128 if prec == "c128" else TOL_C64
    refs = [oracle_lib.contract(net if prec == "c128" else c64_leaves(net), tree) for net, tree, _ in nets]
    for _ in range(3):                                     # replays, with the workspace's old values in place
        outs = batch.contract(leaves, ws)
        torch.cuda.synchronize()
        errs = [rel(o.cpu().numpy(), r) for o, r in zip(outs, refs)]
        note("batch levels", prec, batch.info(), ["%.1e" % e for e in errs])
        assert max(errs) < tol
