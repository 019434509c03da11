"""When a handle's memory is given back: at once, whichever of the matrix and its transpose goes last, without the garbage
collector; and nobody gets it while calls on another stream than the memory's own may still run."""
import gc

import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2403_14853_amd as isp
from paper_2403_14853_amd import autograd as isp_autograd
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


class Busy:
    """Keeps a stream at work for some tenths of a second."""

    def __init__(self, stream):
        with torch.cuda.stream(stream):
            self.keep = torch.zeros(1 << 30, device="cuda")
            for _ in range(300):
                self.keep.mul_(2)
        self.stream = stream

    def still(self):
        return not self.stream.query()


def in_use():
    """Bytes that the allocator cannot hand out, blocks among them that other streams still use."""
    torch.cuda.synchronize()
    torch.empty(1, device="cuda")  # (it looks at what has finished when it is asked)
    return torch.cuda.memory_stats()["active_bytes.all.current"]


def ranges(tensors):
    return [(t.data_ptr(), t.numel() * t.element_size()) for t in tensors if torch.is_tensor(t)]


def given_again(blocks, stream):
    """Which of the blocks the allocator hands out to requests of their sizes on that stream (nothing is written to them)."""
    with torch.cuda.stream(stream):
        got = [torch.empty(n, dtype=torch.uint8, device="cuda") for _, n in sorted(blocks, key=lambda b: -b[1])]
    return [(p, n) for p, n in blocks if any(p < t.data_ptr() + t.numel() and t.data_ptr() < p + n for t in got)]


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("end", ["dropped", "destroyed"])
def test_borrowed_tensors_of_another_stream(graph, transpose, end):
    """As a loader hands them over: copied on a stream of its own, which the computing stream has waited for."""
    indptr, indices, values, _ = graph
    X = torch.from_numpy(graphgen.normal((N, D), 5)).cuda()
    Y = torch.empty_like(X)
    main, copies = torch.cuda.current_stream(), torch.cuda.Stream()
    before = in_use()
    with torch.cuda.stream(copies):
        dev = [torch.from_numpy(a).cuda() for a in (indptr, indices, values)]
    main.wait_stream(copies)
    copies.synchronize()
    A = isp.csr_build(*dev)
    if transpose:
        isp.csr_transpose_cached(A)
    blocks = ranges(dev)
    busy = Busy(main)
    isp.spmm(A, X, Y)
    if end == "destroyed":
        A.destroy()
    del A, dev
    again = given_again(blocks, copies)
    assert busy.still() and not again
    torch.cuda.synchronize()
    assert_close(Y, *oracle.spmm(indptr, indices, values, X.cpu().numpy()))
    del busy
    assert in_use() == before


@pytest.mark.parametrize("how, transpose", [(how, t) for how in ("current", "argument", "autograd", "alias", "alias last") for t in (False, True)] + [("transpose", True)])
def test_calls_on_another_stream(graph, how, transpose):
    X = torch.from_numpy(graphgen.normal((N, D), 5)).cuda()
    Y = torch.empty_like(X)
    main, side = torch.cuda.current_stream(), torch.cuda.Stream()
    before = in_use()
    if how == "autograd":
        G = isp_autograd.SparseGraph(*graph[3])
        A = G.handle
    else:
        A = isp.csr_build(*graph[3])
    if transpose:
        isp.csr_transpose_cached(A)
    blocks = ranges(A._keep[3:])  # the workspaces
    side.wait_stream(main)
    busy = Busy(side)
    if how == "current":
        with torch.cuda.stream(side):
            isp.spmm(A, X, Y)
    elif how == "argument":
        isp.spmm(A, X, Y, stream=side)
    elif how == "transpose":
        isp.spmm(isp.csr_transpose_cached(A)[0], X, Y, stream=side)
    elif how == "autograd":
        with torch.cuda.stream(side):
            out = isp_autograd.spmm(G, X)
        del G
    elif how == "alias":
        B = isp.csr_alias(A)
        isp.spmm(B, X, Y, stream=side)
        blocks += ranges([B._keep[1]])
        del B
    else:  # (the alias is what lets go of its matrix)
        B = isp.csr_alias(A)
        isp.spmm(B, X, Y, stream=side)
        del A
        A = B
        del B
    del A
    again = given_again(blocks, main)
    assert busy.still() and not again
    torch.cuda.synchronize()
    if how == "autograd":
        Y.copy_(out)
        del out
    if how != "transpose":
        assert_close(Y, *oracle.spmm(*graph[:3], X.cpu().numpy()))
    del busy
    assert in_use() == before


@pytest.mark.parametrize("how", ["current", "argument"])
def test_streams_that_torch_did_not_make_leave_it_to_the_collector(graph, how):
    X = torch.zeros(N, D, device="cuda")
    Y = torch.empty_like(X)
    before = allocated()
    A = isp.csr_build(*graph[3])
    isp.csr_transpose_cached(A)
    made = torch.cuda.Stream()
    foreign = torch.cuda.ExternalStream(made.cuda_stream)
    foreign.wait_stream(torch.cuda.current_stream())
    if how == "current":
        with torch.cuda.stream(foreign):
            isp.spmm(A, X, Y)
    else:
        isp.spmm(A, X, Y, stream=foreign)
    torch.cuda.current_stream().wait_stream(foreign)
    held = allocated()
    del A
    assert held >= allocated() > before
    gc.collect()
    assert allocated() == before


def test_handles_used_first_and_dropped_during_a_capture(graph):
    indptr, indices, values, dev = graph
    X = torch.from_numpy(graphgen.normal((N, D), 5)).cuda()
    Y = torch.empty_like(X)
    A, B = isp.csr_build(*dev), isp.csr_build(*dev)
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    other.wait_stream(torch.cuda.current_stream())
    isp.spmm(B, X, torch.empty_like(X), stream=other)
    torch.cuda.synchronize()
    isp.spmm(A, X, Y)
    g = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=side):
        isp.spmm(A, X, Y, stream=side)
        del B
    ref = oracle.spmm(indptr, indices, values, X.cpu().numpy())
    for _ in range(3):
        Y.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert_close(Y, *ref)
        torch.cuda.synchronize()
