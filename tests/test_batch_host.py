"""What a batch of networks (tn_batch) launches, decided on the host."""

import numpy as np
import pytest

from tn_inputs.network import Network, Tree

TWO = Tree(np.array([0], np.int32), np.array([1], np.int32))


def _node(m, n, k):
    M, N, K = list(range(m)), list(range(m, m + n)), list(range(m + n, m + n + k))
    return Network([np.zeros(())] * 2, [M + K, N + K], [2] * (m + n + k), M + N)


@pytest.mark.parametrize("shape,shared", [((5, 5, 4), True), ((5, 5, 6), True), ((5, 5, 7), False), ((6, 6, 8), False),
                                          ((5, 5, 11), False)])
def test_flagged_gemms_keep_their_kernel(shape, shared):
    """TN_FLAG_GEMM_ALL_SIZES sends GEMM-shaped contractions to the matrix
    cores; a batch takes only those of up to 2^16 multiply-adds into its
    shared launch."""
    from paper_2002_01935_amd.binding import Batch, Plan
    plan = Plan(_node(*shape), TWO, gemm_all_sizes=True)
    assert plan.nodes()[0]["kclass"].startswith("gemm")
    assert Batch([plan]).info()["tiny_ops"] == int(shared)
