"""Long sums to few outputs over operands that hold the summed indices in
different orders (splitk_rows_kernel: all rows in one wavefront) against the
oracle: one to eight rows, one to four in-thread outputs, and the shapes next
to the kernel's limits, which keep the ordinary split-K kernel."""

import numpy as np
import pytest

from tests.gpu_util import TOL_C64, TOL_C128, c64_leaves, note, rel, to_dev
from tn_inputs.graphs import pairwise_network
from tn_inputs.network import Tree

pytestmark = pytest.mark.gpu
TWO = Tree(np.array([0], np.int32), np.array([1], np.int32))


@pytest.mark.parametrize("prec", ["c64_4m", "c128"])
@pytest.mark.parametrize("m,n,k,taken", [(1, 0, 18, True), (1, 1, 20, True), (2, 0, 19, True), (2, 1, 18, True),
                                         (2, 2, 19, True), (3, 0, 19, True), (3, 1, 18, True), (3, 2, 19, None),
                                         (0, 0, 18, False), (4, 0, 18, False), (1, 1, 15, False)])
def test_split_rows(oracle_lib, m, n, k, taken, prec):
    import torch

    from paper_2002_01935_amd.binding import Plan
    net = pairwise_network(0, m, n, k, seed=m + 4 * n + 16 * k, dims=(2,))
    plan = Plan(net, TWO, precision=prec)
    kernel = plan.nodes()[0]["kernel"]
    taken = prec != "c128" if taken is None else taken      # 32 complex sums per lane: FP32 only
    assert kernel == ("splitk_rows_kernel" if taken else "splitk_kernel"), kernel
    got = plan.contract(to_dev(net, prec))
    torch.cuda.synchronize()
    e = rel(got.cpu().numpy(), oracle_lib.contract(net if prec == "c128" else c64_leaves(net), TWO))
    note("split rows", (m, n, k), prec, kernel, "%.2e" % e)
    assert e < (TOL_C128 if prec == "c128" else TOL_C64)
