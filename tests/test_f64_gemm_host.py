"""Launch rules of GEMMs, decided on the host: tiles and splits of complex128
ones, splits of the reverse program."""

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


@pytest.mark.parametrize("shape,cap,mib", [((5, 5, 15), 4, 3.0), ((5, 5, 15), 16, 15.2), ((7, 10, 10), 4, 6.0), ((7, 10, 10), 24, 24.0),
                                           ((7, 10, 10), 64, 60.0), ((10, 10, 9), 64, 64.0)])
def test_partial_tiles_stay_within_the_cap(shape, cap, mib):
    """Splits for parallelism take no room from the slices in flight that
    workspace_cap (MiB) asks for: the workspace is `mib`, as many slices as fit
    without the partial tiles."""
    from paper_2002_01935_amd.binding import Plan
    net, S = node(*shape, 4)
    plan = Plan(net, TWO, sliced=S, precision="c128", workspace_cap=cap << 20)
    assert abs(plan.info()["workspace_bytes"] / 2 ** 20 - mib) < 0.1


@pytest.mark.parametrize("shape", [(7, 10, 10), (8, 9, 9), (6, 7, 12), (5, 5, 15)])
def test_partial_tiles_stay_within_the_static_scratch(shape):
    """Nor do they push a plan over the 64 MiB that the call without a
    workspace has: whatever fits without them fits."""
    from paper_2002_01935_amd.binding import Plan
    net, S = node(*shape, 4)
    m, n, k = shape
    hi = max(0, min(k - 9, 9 - max(0, m - 7) - max(0, n - 7)))     # splits that short launches need anyway
    for nb in (1, 2, 3, 4, 6, 8, 12, 16):
        plan = Plan(net, TWO, sliced=S, precision="c128", max_inflight_slices=nb)
        plain = nb * 16 * (2 ** (m + n) + (2 ** (m + n + hi) if hi else 0))
        if plain + 8192 <= 64 << 20:
            assert plan.info()["workspace_bytes"] <= 64 << 20, nb


@pytest.mark.parametrize("prec", ["c64_4m", "c64_3m", "c64_bf16x3"])
def test_reverse_gemms_of_sliced_plans_are_not_split_for_parallelism(prec):
    """Slices in flight fill the chip; an unsliced plan splits its reverse GEMMs
    (the workspace holds their partial tiles), a sliced one does not."""
    from paper_2002_01935_amd.binding import Plan
    net, _ = node(7, 12, 7)
    split = Plan(net, TWO, precision=prec).backward_info([0, 1])["workspace_bytes"]
    net, S = node(7, 12, 7, 2)
    for nb in (1, 4):
        plan = Plan(net, TWO, sliced=S, precision=prec, max_inflight_slices=nb)
        assert plan.backward_info([0, 1])["workspace_bytes"] < nb * split
