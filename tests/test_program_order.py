"""The planner's forward and reverse programs, with the small contractions
collected into group launches, run op by op on the host
(tests/emu/emu_program.cpp) against the oracle: every value is written before
an op reads it and keeps its memory until its last reader, whatever the order
of the launches."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from tn_inputs.graphs import random_network
from tn_inputs.greedy import find_tree
from tn_inputs.network import Network, Tree

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
PREC = {"c64_4m": 0, "c128": 3}
# the arithmetic is in double, values are stored in the plan's type: products
# of tens of float32 roundings (6e-8 each), or of double ones
TOL = {"c64_4m": 1e-5, "c128": 1e-12}


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if not os.path.exists(CLANG) and shutil.which("clang++") is None:
        pytest.skip("no clang++ for the host build")
    cxx = CLANG if os.path.exists(CLANG) else shutil.which("clang++")
    out = str(tmp_path_factory.mktemp("emu") / "emu_program")
    csrc = os.path.join(ROOT, "paper_2002_01935_amd", "csrc")
    subprocess.run([cxx, "-O2", "-std=c++20", "-I", csrc, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "emu", "emu_program.cpp"), os.path.join(csrc, "plan.cpp"), "-o", out,
                    "-lpthread"], check=True, capture_output=True)
    return out


def describe(d, net, tree, sliced, ids, wrt, opt):
    lists = [[len(t) for t in net.leaf_idx], [i for t in net.leaf_idx for i in t], list(net.idx_dim), list(net.out_idx),
             list(tree.left), list(tree.right), list(sliced), list(ids), list(wrt), opt]
    with open(os.path.join(d, "net.txt"), "w") as f:
        for x in lists:
            f.write(" ".join(str(int(v)) for v in [len(x)] + x) + "\n")


def run(emu, d, net, tree, prec, wrt, go, sliced=(), ids=(0,), grouped=True):
    describe(d, net, tree, sliced, ids, wrt, [PREC[prec], 0, int(grouped)])
    with open(os.path.join(d, "in.bin"), "wb") as f:
        for t in list(net.leaves) + [go]:
            np.ascontiguousarray(t, dtype=np.complex128).tofile(f)
    r = subprocess.run([emu, os.path.join(d, "net.txt"), os.path.join(d, "in.bin"), os.path.join(d, "out.bin")],
                       capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    flat = np.fromfile(os.path.join(d, "out.bin"), dtype=np.complex128)
    shapes = [tuple(net.idx_dim[e] for e in net.out_idx)] + [np.shape(net.leaves[v]) for v in wrt]
    out, at = [], 0
    for s in shapes:
        n = int(np.prod(s, dtype=np.int64))
        out.append(flat[at:at + n].reshape(s))
        at += n
    assert at == len(flat)
    return out[0], out[1:]


def check(emu, oracle_lib, tmp_path, net, tree, wrt, precs=PREC, sliced=(), ids=(0,), seed=0):
    rng = np.random.default_rng(seed)
    shape = tuple(net.idx_dim[e] for e in net.out_idx)
    go = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    ref = oracle_lib.contract(net, tree, sliced=list(sliced), slice_ids=list(ids))
    refs = oracle_lib.grad(net, tree, go, wrt, sliced=list(sliced), slice_ids=list(ids))
    for prec in precs:
        got, grads = run(emu, str(tmp_path), net, tree, prec, wrt, go, sliced, ids)
        for g, r in zip([got] + grads, [ref] + refs):
            assert np.linalg.norm(np.ravel(g) - np.ravel(r)) <= TOL[prec] * np.linalg.norm(np.ravel(r)), prec


def forked_group():
    """(((L1 L2) l2) l3) w) u with wrt = {3, 5}: in the reverse program one
    connected set of small contractions holds both a forward value that a large
    contraction reads and, further on, a cotangent that needs a later large one."""
    a, m = list(range(11)), list(range(18, 30))
    i1, i2, j1, j2, k1, k2, z = 11, 12, 13, 14, 15, 16, 17
    idx = [a + [i1, i2], a + [j1, j2], [i1, k1], [i2, k2], [k1] + m, [k2, z]]
    rng = np.random.default_rng(3)
    leaves = [(rng.normal(size=(2,) * len(t)) + 1j * rng.normal(size=(2,) * len(t))) for t in idx]
    net = Network(leaves, idx, [2] * 30, [j1, j2, z] + m)
    net.check()
    return net, Tree(np.array([0, 6, 7, 8, 9], np.int32), np.array([1, 2, 3, 4, 5], np.int32))


# (leaves, largest rank, outputs, graph): random networks whose reverse
# programs hold such a group, and others
GRAPHS = [(21, 5, 5, 57), (16, 6, 4, 34881), (19, 5, 5, 99433), (24, 6, 6, 23629), (25, 4, 5, 51936), (36, 5, 6, 21123),
          (14, 5, 3, 1), (22, 4, 4, 2), (30, 5, 3, 3), (40, 4, 2, 4)]


def random_case(leaves, rank, n_out, graph):
    net = random_network(leaves, 7 * leaves // 5, rank, graph, n_out=n_out, dims=(2, 4), hyper=True)
    return net, find_tree(net, seed=0, trials=1)


def test_reader_of_a_group_that_waits_for_a_later_op(emu, oracle_lib, tmp_path):
    net, tree = forked_group()
    check(emu, oracle_lib, tmp_path, net, tree, [3, 5])


@pytest.mark.parametrize("case", GRAPHS)
def test_random_programs(emu, oracle_lib, tmp_path, case):
    net, tree = random_case(*case)
    check(emu, oracle_lib, tmp_path, net, tree, list(range(net.n_leaves)))


def test_random_program_sliced(emu, oracle_lib, tmp_path):
    net, tree = random_case(*GRAPHS[0])
    sliced = [e for e in range(net.n_idx) if e not in net.out_idx][:3]
    check(emu, oracle_lib, tmp_path, net, tree, list(range(net.n_leaves)), sliced=sliced, ids=(0, 3, 5))


def chain(length, dim):
    """A vector times `length` - 1 matrices of dim x dim, one after another."""
    idx = [[0]] + [[v - 1, v] for v in range(1, length)]
    left = [0] + [length + v for v in range(length - 2)]
    return idx, [dim] * length, [length - 1], Tree(np.array(left, np.int32), np.array(range(1, length), np.int32))


@pytest.mark.parametrize("length,dim", [(400, 2), (700, 4), (40, 32)])
def test_chains_cut_into_groups(emu, oracle_lib, tmp_path, length, dim):
    """Connected sets of more contractions than one group takes, or than LDS holds."""
    idx, dims, out, tree = chain(length, dim)
    rng = np.random.default_rng(length)
    leaves = [(rng.normal(size=(dim,) * len(t)) + 1j * rng.normal(size=(dim,) * len(t))) / (1.4 * dim ** 0.5) for t in idx]
    check(emu, oracle_lib, tmp_path, Network(leaves, idx, dims, out), tree, list(range(0, length, 7)))


def test_planning_time_of_long_chains():
    """16,000 contractions in one connected set: planned in seconds, forward and
    reverse (0.3 + 1 s; cutting one group per pass took 5 + 13 s)."""
    import time

    from paper_2002_01935_amd.binding import Plan
    idx, dims, out, tree = chain(16000, 4)
    t0 = time.perf_counter()
    Plan(Network([None] * len(idx), idx, dims, out), tree).backward_info(list(range(0, 16000, 5)))
    assert time.perf_counter() - t0 < 6


def row_ops(emu, tmp_path, net, tree, sliced, wrt, prec, inflight):
    """(reverse, log2 rows, in-thread outputs, summed values, chunks or -1) of every row and split-K contraction."""
    describe(str(tmp_path), net, tree, sliced, (0,), wrt, [PREC[prec], 0, 0, inflight])
    out = subprocess.run([emu, str(tmp_path / "net.txt"), "-", "-"], capture_output=True, text=True, check=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def _chain(k, ks):
    """Additions a value passes: its lane's, then the chunks' (64 lanes and a butterfly)."""
    return 2 ** (k - 6 - ks) + (2 ** (ks - 6) + 6 if ks > 6 else ks)


@pytest.mark.parametrize("prec", PREC)
@pytest.mark.parametrize("m,n", [(0, 0), (1, 0), (1, 1), (2, 1), (3, 2), (5, 2), (8, 4), (10, 0), (10, 4), (13, 0)])
def test_length_of_split_sums(emu, tmp_path, m, n, prec):
    """A split sum in any program passes at most the additions that 2^15
    wavefronts (rows x chunks) give it, whatever order the operands hold the
    summed bits in."""
    seen = 0
    for k in range(6, 30):
        if m + k > 30:
            break
        M, N, K = list(range(m)), list(range(m, m + n)), list(range(m + n, m + n + k))
        z = m + n + k
        for order in (K, K[::-1]):
            # node 1 = A B, then a vector: the reverse program sums node 1 again
            net = Network([np.zeros(())] * 3, [M + K, N + order, [z]], [2] * (z + 1), M + N + [z])
            tree = Tree(np.array([0, 3], np.int32), np.array([1, 2], np.int32))
            for rev, _, _, kk, ks in row_ops(emu, tmp_path, net, tree, (), [2], prec, 1):
                if kk != k or ks < 0:
                    continue
                most = min(k - 6, max(0, 15 - (m + n - min(4, min(m, n)))))
                most2 = min(k - 6, max(0, 15 - (m + n - min(4, max(m, n)))))
                assert _chain(k, ks) <= max(_chain(k, most), _chain(k, most2)), (rev, m, n, k, ks)
                seen += 1
    assert seen > 20


@pytest.mark.parametrize("prec", PREC)
@pytest.mark.parametrize("m,k,slices,inner", [(12, 5, 0, 0), (12, 5, 1, 1), (12, 5, 4, 4), (12, 5, 6, 4), (8, 5, 0, 0), (8, 5, 6, 2),
                                              (8, 10, 0, 4), (5, 9, 0, 0), (5, 9, 2, 2), (5, 9, 6, 4), (16, 5, 0, 4)])
def test_outputs_per_thread(emu, tmp_path, m, k, slices, inner, prec):
    """2^m rows x 16 outputs: as few of the 16 stay in one thread as fill the
    chip with the slices in flight (2^16 threads, or 2^12 wavefronts of split
    sums), all of them where the rows do."""
    M, N, K, S = [list(range(*r)) for r in ((0, m), (m, m + 4), (m + 4, m + 4 + k), (m + 4 + k, m + 4 + k + slices))]
    net = Network([np.zeros(())] * 2, [S + M + K, S + N + K], [2] * (m + 4 + k + slices), M + N)
    ops = row_ops(emu, tmp_path, net, Tree(np.array([0], np.int32), np.array([1], np.int32)), S, [], prec, 2 ** slices)
    assert [(op[1], op[2]) for op in ops] == [(m + 4 - inner, inner)]


@pytest.mark.gpu
@pytest.mark.parametrize("prec", PREC)
@pytest.mark.parametrize("case", [None] + GRAPHS[:6])
def test_gradients_on_the_gpu(oracle_lib, case, prec):
    import torch

    from paper_2002_01935_amd.binding import Plan
    from tests.gpu_util import TOL_C64, TOL_C128, note, ref_net, rel, to_dev
    net, tree = forked_group() if case is None else random_case(*case)
    wrt = [3, 5] if case is None else list(range(net.n_leaves))
    rng = np.random.default_rng(0)
    shape = tuple(net.idx_dim[e] for e in net.out_idx)
    go = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    grads = Plan(net, tree, precision=prec).backward(to_dev(net, prec), torch.from_numpy(go), wrt)
    torch.cuda.synchronize()
    refs = oracle_lib.grad(ref_net(net, prec), tree, go, wrt)
    worst = max(rel(g.cpu().numpy(), r) for g, r in zip(grads, refs))
    note("gradients, program order", case, prec, "%.2e" % worst)
    assert worst < (TOL_C128 if prec == "c128" else TOL_C64)
