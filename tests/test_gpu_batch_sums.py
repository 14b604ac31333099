"""Long sums in a batch of networks (tn_batch): their rounding error, and the
sums that are left to the split-K kernels."""

import numpy as np
import pytest

from tests.gpu_util import note
from tn_inputs.network import Network, Tree

pytestmark = pytest.mark.gpu
TWO = Tree(np.array([0], np.int32), np.array([1], np.int32))


def _sums(n_out, k, count, dtype):
    """`count` contractions A(M, K) x B(N, K) -> (M, N) of 2^n_out outputs and
    2^k random complex products each, their leaves on the GPU and their values
    in double precision."""
    import torch
    m = n_out // 2
    M, N, K = list(range(m)), list(range(m, n_out)), list(range(n_out, n_out + k))
    real = torch.float64 if dtype == torch.complex128 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(100 * n_out + k)
    shape_only = Network([np.zeros((1,) * 0)] * 2, [M + K, N + K], [2] * (n_out + k), M + N)
    nets, leaves, refs = [], [], []
    for _ in range(count):
        a, b = [torch.complex(*[torch.randn(2 ** (x + k), generator=gen, device="cuda", dtype=real) for _ in range(2)])
                for x in (m, n_out - m)]
        nets.append(shape_only)
        leaves.append([a, b])
        A, B = a.to(torch.complex128).reshape(-1, 2 ** k), b.to(torch.complex128).reshape(-1, 2 ** k)
        refs.append(torch.stack([(A[i] * B).sum(-1) for i in range(A.shape[0])]).ravel())
    return nets, leaves, refs


@pytest.mark.parametrize("n_out,k", [(0, 6), (0, 12), (0, 16), (4, 14), (8, 12), (10, 12), (9, 13), (14, 7), (16, 6), (15, 6),
                                     (0, 17), (0, 18), (0, 22), (5, 17)])
def test_error_of_long_sums(n_out, k):
    """A balanced tree of additions: every value passes k of them, so the error
    relative to the terms' root-sum-square, 2^(k / 2) products of rms 2, is at
    most about 2^-24 sqrt(k + 3) (a product and its conversion counted as three
    more; roundings independent, each up to 2^-24 of a partial sum that grows
    as the root of its length).  Sums above 2^16 values run the kernels that
    Plan.contract runs: the same bits."""
    import torch

    from paper_2002_01935_amd.binding import Batch, Plan
    count = 16 if n_out < 9 else 2
    nets, leaves, refs = _sums(n_out, k, count, torch.complex64)
    plans = [Plan(net, TWO) for net in nets]
    batch = Batch(plans)
    ws = batch.workspace()
    batch.prepare(ws)
    assert batch.info()["launches"] == (1 if k <= 16 else 2 * count)
    for _ in range(2):
        outs = batch.contract(leaves, ws)
    alone = [p.contract(ls) for p, ls in zip(plans, leaves)]
    torch.cuda.synchronize()
    err = torch.cat([o.ravel().to(torch.complex128) - r for o, r in zip(outs, refs)]).abs().square().mean().sqrt().item()
    err /= 2.0 * 2.0 ** (k / 2)
    bound = 2.0 ** -24 * np.sqrt(k + 3)
    note("long sums", n_out, k, "error %.2e, bound %.2e" % (err, bound))
    if k <= 16:
        assert err < bound
    else:
        assert all(torch.equal(o, a) for o, a in zip(outs, alone))
