"""complex128 GEMMs on the FP64 matrix cores (gemm_mfma_f64) against the
oracle: partial and full tiles of the three block shapes, batch bits, shuffled
operand and output orders, few and many summed values, sums split over the
grid, and conjugated operands (reverse mode)."""

import numpy as np
import pytest

from tests.gpu_util import TOL_C128, note, rel, to_dev
from tn_inputs.graphs import pairwise_network
from tn_inputs.network import Tree

pytestmark = pytest.mark.gpu
TWO = Tree(np.array([0], np.int32), np.array([1], np.int32))

# (h, m, n, k), kernel, split over K; the oracle's work stays under 2^27 products
SHAPES = [((0, 5, 5, 4), "32,64", False), ((0, 5, 9, 5), "32,64", False), ((2, 6, 7, 4), "32,64", False),
          ((0, 7, 6, 8), "32,64", True), ((1, 6, 6, 11), "32,64", True), ((0, 8, 5, 10), "32,64", True),
          ((3, 5, 6, 9), "32,64", True), ((0, 11, 11, 4), "128,64", False), ((4, 9, 9, 4), "128,64", False),
          ((0, 12, 10, 5), "128,64", False), ((0, 10, 11, 4), "64,64", False), ((3, 9, 9, 5), "64,64", False),
          ((0, 10, 10, 6), "32,64", False)]


@pytest.mark.parametrize("shape,kernel,split", SHAPES, ids=["-".join(map(str, s[0])) for s in SHAPES])
def test_f64_gemm(oracle_lib, shape, kernel, split):
    import torch

    from paper_2002_01935_amd.binding import Plan
    net = pairwise_network(*shape, seed=sum(shape))
    plan = Plan(net, TWO, precision="c128", gemm_all_sizes=True)
    node = plan.nodes()[0]
    assert node["kernel"].startswith(f"gemm_mfma_f64<{kernel}"), node
    assert (node["kclass"] == "gemm_splitk") == split, node
    leaves = to_dev(net, "c128")
    got = plan.contract(leaves)
    torch.cuda.synchronize()
    e = rel(got.cpu().numpy(), oracle_lib.contract(net, TWO))
    note("f64 gemm", shape, node["kernel"], "%.2e" % e)
    assert e < TOL_C128
    if sum(shape) <= 22:
        rng = np.random.default_rng(sum(shape))
        oshape = tuple(net.idx_dim[i] for i in net.out_idx)
        go = rng.normal(size=oshape) + 1j * rng.normal(size=oshape)
        refs = oracle_lib.grad(net, TWO, go, [0, 1])
        grads = plan.backward(leaves, torch.from_numpy(go), [0, 1])
        torch.cuda.synchronize()
        for g, r in zip(grads, refs):
            assert rel(g.cpu().numpy(), r) < TOL_C128
