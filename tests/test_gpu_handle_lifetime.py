"""When a handle's workspaces are given back: at once, whichever of the matrix and its transpose goes last, without the garbage
collector; but not while calls on another stream than the workspaces' own may still run."""
import gc

import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close

pytestmark = pytest.mark.gpu

N, D = 3000, 20


@pytest.fixture
def graph():
    indptr, indices = graphgen.rmat_graph(N, 40_000, seed=3)
    values = graphgen.uniform(indices.shape[0], 4)
    gc.collect()
    gc.disable()
    yield indptr, indices, values, [torch.from_numpy(a).cuda() for a in (indptr, indices, values)]
    gc.enable()
    gc.collect()


def allocated():
    torch.cuda.synchronize()
    return torch.cuda.memory_allocated()


@pytest.mark.parametrize("last", ["matrix", "transpose"])
def test_workspaces_are_given_back_at_once(graph, last):
    indptr, indices, values, dev = graph
    X = torch.from_numpy(graphgen.normal((N, D), 5)).cuda()
    Y = torch.empty_like(X)
    before = allocated()
    A = isp.csr_build(*dev)
    At, _ = isp.csr_transpose_cached(A)
    assert isp.csr_transpose_cached(A) == (At, True)
    held = allocated()
    assert held > before
    if last == "matrix":
        del At
    else:
        del A
    assert allocated() == held
    if last == "transpose":  # still usable: it keeps what it borrows
        isp.spmm(At, X, Y)
        ti, tj, _, tv = oracle.transpose(N, N, indptr, indices, values)
        assert_close(Y, *oracle.spmm(ti, tj, tv, X.cpu().numpy()))
        del At
    else:
        isp.spmm(A, X, Y)
        assert_close(Y, *oracle.spmm(indptr, indices, values, X.cpu().numpy()))
        del A
    assert allocated() == before


def test_destroyed_matrices_take_their_transpose_along(graph):
    before = allocated()
    A = isp.csr_build(*graph[3])
    At, _ = isp.csr_transpose_cached(A)
    A.destroy()
    A.destroy()
    X = torch.zeros(N, D, device="cuda")
    for h in (A, At):
        with pytest.raises(isp.IspError):
            isp.spmm(h, X, torch.empty_like(X))
    del A, At, X, h
    gc.collect()  # (what the errors remember)
    assert allocated() == before


@pytest.mark.parametrize("how", ["current", "argument", "alias"])
def test_other_streams_leave_it_to_the_collector(graph, how):
    X = torch.zeros(N, D, device="cuda")
    Y = torch.empty_like(X)
    before = allocated()
    A = isp.csr_build(*graph[3])
    isp.csr_transpose_cached(A)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    if how == "current":
        with torch.cuda.stream(side):
            isp.spmm(A, X, Y)
    elif how == "argument":
        isp.spmm(isp.csr_transpose_cached(A)[0], X, Y, stream=side)
    else:
        B = isp.csr_alias(A)
        isp.spmm(B, X, Y, stream=side)
        del B
    torch.cuda.current_stream().wait_stream(side)
    held = allocated()
    del A
    assert held >= allocated() > before
    gc.collect()
    gc.collect()  # (an alias lets go of its matrix in the first)
    assert allocated() == before
