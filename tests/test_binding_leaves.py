"""Leaf lists of the Python binding: what is accepted and what is refused, with
and without the native checks.  No GPU: the checks only read attributes."""

import numpy as np
import pytest
import torch

from tn_inputs.network import Network, Tree

TWO = Tree(np.array([0], np.int32), np.array([1], np.int32))


@pytest.fixture(params=[True, False], ids=["native", "python"])
def B(request, monkeypatch):
    from paper_2002_01935_amd import binding
    assert binding._leaves is not None
    if not request.param:
        monkeypatch.setattr(binding, "_leaves", None)
    return binding


class Like:
    """An object with a CUDA tensor's attributes."""
    is_cuda, dtype, shape = True, torch.complex64, (2, 2)

    def __init__(self, address, **changes):
        self.address = address
        self.__dict__.update(changes)

    def is_contiguous(self):
        return True

    def numel(self):
        return int(np.prod(self.shape))

    def data_ptr(self):
        return self.address


def _plan(B):
    return B.Plan(Network([np.zeros((2, 2))] * 2, [[0, 1], [1, 2]], [2, 2, 2], [0, 2]), TWO)


def test_objects_like_tensors(B):
    p = _plan(B)
    assert bytes(p._check_leaves([Like(4096), Like(8192)])) == np.array([4096, 8192], np.uint64).tobytes()
    assert bytes(p._check_leaves({0: Like(4096), 1: Like(8192)}.values())) == np.array([4096, 8192], np.uint64).tobytes()
    for bad in (dict(is_cuda=False), dict(dtype=torch.complex128), dict(shape=(2, 4))):
        with pytest.raises(ValueError, match="leaf 1"):
            p._check_leaves([Like(4096), Like(8192, **bad)])


def test_refused_leaves(B):
    p = _plan(B)
    cpu = torch.zeros(2, 2, dtype=torch.complex64)
    for leaves in ([cpu, cpu], (cpu, cpu), torch.zeros(2, 2, 2, dtype=torch.complex64), {0: cpu, 1: cpu}.values()):
        with pytest.raises(ValueError, match="leaf 0 must be a contiguous"):
            p._check_leaves(leaves)
    with pytest.raises(ValueError, match="expected 2 leaves"):
        p._check_leaves([cpu])
    with pytest.raises(AttributeError):
        p._check_leaves([np.zeros((2, 2)), np.zeros((2, 2))])


def test_leaf_beyond_64_bits_is_refused_by_the_planner(B):
    K = list(range(70))
    with pytest.raises(B.TNError) as e:
        B.Plan(Network([np.zeros(())] * 2, [K, K], [2] * 70, []), TWO)
    assert e.value.code in (-1, -2)
