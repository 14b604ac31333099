"""Launch rules of the complex128 GEMMs, decided on the host."""

import numpy as np
import pytest

from tn_inputs.network import Network, Tree

TWO = Tree(np.array([0], np.int32), np.array([1], np.int32))


def node(m, n, k, slices=0):
    """A(S, M, K) x B(S, N, K) -> (M, N), the `slices` bits of S sliced."""
    M, N, K, S = [list(range(*r)) for r in ((0, m), (m, m + n), (m + n, m + n + k), (m + n + k, m + n + k + slices))]
    return Network([np.zeros(())] * 2, [S + M + K, S + N + K], [2] * (m + n + k + slices), M + N), S


@pytest.mark.parametrize("shape,slices,tile", [((8, 10, 8), 0, "<32,64"), ((8, 10, 8), 6, "<128,64"), ((9, 9, 9), 0, "<32,64"),
                                               ((9, 9, 9), 6, "<128,64"), ((12, 12, 8), 0, "<128,64")])
def test_tile_counts_the_slices_in_flight(shape, slices, tile):
    """Small tiles where a launch has few blocks: those of all slices in flight."""
    from paper_2002_01935_amd.binding import Plan
    net, S = node(*shape, slices)
    plan = Plan(net, TWO, sliced=S, precision="c128", max_inflight_slices=2 ** slices)
    assert tile in plan.nodes()[0]["kernel"]
