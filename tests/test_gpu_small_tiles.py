"""The 64 x 64 block tiles of the 4M matrix-core kernels (direct-to-LDS and
register-staged, four waves of 32 x 32) against the oracle and, bit for bit,
against the 128 x 128 tile of the same kernel: partial tiles, batch bits,
summed ranges from one pipeline stage on, sums split over the grid."""

import numpy as np
import pytest

from tests.gpu_util import TOL_C64, c64_leaves, note, rel, to_dev
from tn_inputs.graphs import pairwise_network
from tn_inputs.network import Network, Tree

pytestmark = pytest.mark.gpu
TWO = Tree(np.array([0], np.int32), np.array([1], np.int32))
SHAPES = [(0, 5, 5, 4), (0, 6, 6, 4), (2, 5, 7, 5), (0, 7, 6, 6), (0, 6, 9, 4), (0, 8, 8, 5), (1, 6, 5, 11)]


def _canonical(h, m, n, k, rng):
    """Operands A[h, m, k] and B[h, n, k]: summed indices lowest, as the planner lays intermediates out."""
    H, M, N, K = (list(range(s, s + c)) for s, c in ((0, h), (h, m), (h + m, n), (h + m + n, k)))
    idx = [H + M + K, H + N + K]
    leaves = [rng.normal(size=(2,) * len(ix)) + 1j * rng.normal(size=(2,) * len(ix)) for ix in idx]
    return Network(leaves, idx, [2] * (h + m + n + k), H + M + N)


@pytest.mark.parametrize("layout,small,large", [("canonical", 15, 9), ("shuffled", 16, 0)])
@pytest.mark.parametrize("shape", SHAPES, ids=["-".join(map(str, s)) for s in SHAPES])
def test_small_tiles(oracle_lib, shape, layout, small, large):
    import torch

    from paper_2002_01935_amd.binding import Plan
    rng = np.random.default_rng(sum(shape))
    net = _canonical(*shape, rng) if layout == "canonical" else pairwise_network(*shape, seed=sum(shape), dims=(2,))
    plan = Plan(net, TWO, precision="c64_4m", gemm_all_sizes=True)
    assert plan.nodes()[0]["tile"] == small, plan.nodes()   # fewer than two large blocks per compute unit
    leaves = to_dev(net, "c64_4m")
    got = plan.contract(leaves)
    assert plan.set_tile(large) == 1
    wide = plan.contract(leaves)
    torch.cuda.synchronize()
    e = rel(got.cpu().numpy(), oracle_lib.contract(c64_leaves(net), TWO))
    note("small tile", shape, layout, "%.2e" % e)
    assert e < TOL_C64
    assert torch.equal(torch.view_as_real(got), torch.view_as_real(wide))
