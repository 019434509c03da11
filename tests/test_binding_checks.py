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


def test_tensors_without_storage_raise(nat, cell):
    """vmap's tensors have no storage to point into: an exception, in every entry point."""
    from torch._subclasses.fake_tensor import FakeTensorMode
    graph = nat.graph(cell, object(), None)
    calls = [lambda x: nat.spmm(cell, x, x, 0), lambda x: nat.spmm_static_scratch(cell, x, x, 0),
             lambda x: nat.sddmm(cell, x, x, x, 0, 0), lambda x: nat.fusedmm(cell, x, x, 0, 0),
             lambda x: nat.fusedmm_backward(cell, x, x, x, 0, 0), lambda x: nat.spmm_reduce(cell, x, x, 3, x, 0),
             lambda x: nat.spmm_reduce_backward(cell, x, x, 3, x, 0), lambda x: nat.ag_spmm(graph, None, x),
             lambda x: nat.ag_reduce(graph, x, 3), lambda x: nat.ag_fused(graph, x)]
    with FakeTensorMode():
        X = torch.empty(3, 4, 8, device="cuda")
        for call in calls:
            with pytest.raises(RuntimeError):
                torch.func.vmap(call)(X)


def test_release_looks_at_its_arguments(nat, cell):
    nat.cells_release([cell], [torch.zeros(3), None, object()], None)  # (no call has run on a stream)
    nat.cells_release([cell, cell], [], cell)
    for bad in (lambda: nat.cells_release(cell, [], None), lambda: nat.cells_release([cell], (), None), lambda: nat.cells_release([1], [], None),
                lambda: nat.cells_release([cell], [], 1), lambda: nat.cells_release([cell], []), lambda: nat.cell_ran(cell, "x"), lambda: nat.cell_foreign(None)):
        with pytest.raises((AssertionError, TypeError, ValueError)):
            bad()


def test_forward_mode_is_refused(nat, cell):
    import torch.autograd.forward_ad as fw
    graph = nat.graph(cell, object(), None)
    t = torch.zeros(4, 8)
    with fw.dual_level():
        x = fw.make_dual(t, torch.ones(4, 8))
        v = fw.make_dual(torch.ones(6), torch.ones(6))
        for call in (lambda: nat.ag_spmm(graph, None, x), lambda: nat.ag_spmm(graph, v, t),
                     lambda: nat.ag_reduce(graph, x, 3), lambda: nat.ag_fused(graph, x)):
            with pytest.raises(NotImplementedError):
                call()
        with fw._set_fwd_grad_enabled(False), pytest.raises(AssertionError):  # (not a tangent then; refused as a CPU tensor)
            nat.ag_spmm(graph, None, x)
