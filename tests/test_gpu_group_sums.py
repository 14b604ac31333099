"""Rounding error of the longest sums that a group of small contractions takes
(tiny_tree_kernel), against the same sums in the split-K kernel."""

import numpy as np
import pytest

from tests.gpu_util import note
from tn_inputs.network import Network, Tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [6, 8, 9, 10])
def test_error_of_shared_sums(k):
    """A(K) B(K) x(z) -> (z): the reverse program for x computes the sum over
    2^k values inside a group, Plan.contract on A and B in the split-K kernel.
    In both a value passes k additions, so their rms errors over 4000 random
    sums agree within the statistics (1 % each, three deviations)."""
    import torch

    from paper_2002_01935_amd.binding import Plan
    K = list(range(k))
    zero = np.zeros(())
    net = Network([zero] * 3, [K, K, [k]], [2] * (k + 1), [k])
    grad = Plan(net, Tree(np.array([0, 3], np.int32), np.array([1, 2], np.int32)))
    assert grad.backward_kernels([2]).count("tiny_tree_kernel") >= 2
    alone = Plan(Network([zero] * 2, [K, K], [2] * k, []), Tree(np.array([0], np.int32), np.array([1], np.int32)))
    assert alone.nodes()[0]["kernel"] == "splitk_kernel"
    gen = torch.Generator(device="cuda").manual_seed(k)
    count = 4000
    ab = torch.complex(*[torch.randn(count, 2, 2 ** k, generator=gen, device="cuda") for _ in range(2)])
    x = torch.ones(2, dtype=torch.complex64, device="cuda")
    go = torch.ones(2, dtype=torch.complex128, device="cuda")
    exact = ab[:, 0].to(torch.complex128).mul(ab[:, 1].to(torch.complex128)).sum(-1)
    grads = torch.empty(count, 2, dtype=torch.complex64, device="cuda")
    vals = torch.empty(count, dtype=torch.complex64, device="cuda")
    ws, ws2 = grad.workspace(grad.backward_info([2])["workspace_bytes"]), alone.workspace()
    for i in range(count):
        grad.backward([ab[i, 0], ab[i, 1], x], go, [2], grads=[grads[i]], workspace=ws)
        alone.contract([ab[i, 0], ab[i, 1]], out=vals[i], workspace=ws2)
    torch.cuda.synchronize()
    rms = [(v.to(torch.complex128) - exact).abs().square().mean().sqrt().item() for v in (grads[:, 0].conj(), vals)]
    note("group sums", k, "rms error %.3e, split-K kernel %.3e, ratio %.3f" % (rms[0], rms[1], rms[0] / rms[1]))
    assert rms[0] < 1.05 * rms[1]
