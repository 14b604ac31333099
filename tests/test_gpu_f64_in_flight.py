"""complex128 values do not depend on the slices in flight, bit for bit: the
sum over a GEMM's splits is the same whether the partial tiles go through the
workspace or, where the slices in flight fill the chip or the workspace has no
room, are added inside the kernel."""

import pytest

from tests.gpu_util import note
from tests.test_f64_gemm_host import TWO, node

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(7, 10, 10), (8, 9, 9), (6, 7, 12), (5, 5, 15), (5, 11, 10), (7, 7, 13)])
def test_split_sums_in_and_outside_the_kernel(shape):
    import torch

    from paper_2002_01935_amd.binding import Plan
    m, n, k = shape
    net, S = node(m, n, k, 4)
    gen = torch.Generator(device="cuda").manual_seed(sum(shape))
    a, b = [torch.complex(*[torch.randn(2 ** (4 + x + k), generator=gen, device="cuda", dtype=torch.float64) for _ in range(2)])
            for x in (m, n)]
    ref = sum(a.reshape(16, 2 ** m, 2 ** k)[s] @ b.reshape(16, 2 ** n, 2 ** k)[s].T for s in range(16)).ravel()
    vals, kernels = [], []
    for nb in (1, 2, 3, 4, 6, 8, 12, 16):
        plan = Plan(net, TWO, sliced=S, precision="c128", max_inflight_slices=nb)
        vals.append(plan.contract_sliced([a, b]).ravel())
        kernels.append(plan.nodes()[0]["kernel"])
    torch.cuda.synchronize()
    err = ((vals[0] - ref).norm() / ref.norm()).item()
    note("split sums", shape, "rel err %.1e" % err, kernels)
    assert err < 1e-13
    assert all(torch.equal(v, vals[0]) for v in vals)
    assert {"fold" in x for x in kernels} == {False, True}
