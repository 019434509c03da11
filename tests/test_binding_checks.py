"""What the native binding refuses, on the CPU: arguments are looked at before any library call, so a handle of no matrix
does."""
import numpy as np
import pytest
import torch

from paper_2403_14853_amd import binding


@pytest.fixture(scope="module")
def nat():
    return binding._native()


@pytest.fixture(scope="module")
def cell(nat):
    return nat.cell(0, 4, 4, 6)  # a NULL handle of a 4 x 4 matrix


NOT_TENSORS = [None, np.zeros((4, 8), np.float32), [[1.0, 2.0]], "x", 3.0]


@pytest.mark.parametrize("x", NOT_TENSORS, ids=lambda x: type(x).__name__)
def test_dense_operands_must_be_tensors(nat, cell, x):
    graph = nat.graph(cell, object(), None)
    t = torch.zeros(4, 8)
    for call in (lambda: nat.ag_spmm(graph, None, x), lambda: nat.ag_reduce(graph, x, 3), lambda: nat.ag_fused(graph, x),
                 lambda: nat.spmm(cell, x, t, 0), lambda: nat.spmm_static_scratch(cell, x, t, 0)):
        with pytest.raises(TypeError):
            call()
    if x is not None:  # (None: all ones)
        with pytest.raises(TypeError):
            nat.ag_spmm(graph, x, t)
        with pytest.raises(TypeError):
            nat.graph(cell, object(), x)
