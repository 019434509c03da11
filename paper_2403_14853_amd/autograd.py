"""Thin autograd wrappers over the C ABI, so the sparse operations can sit
inside an ordinary PyTorch training step (the role of the paper's C++ wrapper that connects
forward and backward propagation to the kernels, Section 3.1).  Everything numerical still runs
in the library's HIP kernels; the nodes (csrc/torch_native.cpp) only route tensors and remember what
backward needs.

``SparseGraph`` owns the handle; its transpose is built on the first backward and cached in the
handle for all later epochs (Section 3.3).
"""
from __future__ import annotations

import torch

from . import binding as _b

_recorder = torch._C._get_tracing_state  # None unless torch.jit.trace is recording


class SparseGraph:
    """A CSR matrix on the GPU plus its library handle.  ``values`` may be a leaf tensor that
    requires grad; its gradient is the SDDMM of (dY, X)."""

    def __init__(self, indptr, indices, values=None, n_cols=None):
        self.indptr, self.indices, self.values = indptr, indices, values
        self.handle = _b.csr_build(indptr, indices, None if values is None else values.detach(), n_cols=n_cols)
        self.n_rows, self.n_cols, self.nnz = self.handle.n_rows, self.handle.n_cols, self.handle.nnz
        self._native = _b._native().graph(self.handle._cell, self.handle, values)

    def sync_values(self):
        """The handle reads ``values``' storage directly.  When an optimizer step has rewritten it in place
        since the last call, the arrays derived from it have to pick the new values up (the transpose's structure,
        permutation and partition stay cached).  The operations below do this themselves."""
        _b._native().graph_sync(self._native)

    def transpose(self):
        self.sync_values()
        return _b.csr_transpose_cached(self.handle)[0]


class _Recorded(torch.autograd.Function):
    """One of the operations below while torch.jit.trace records a program: the native nodes are not among the operations
    that a recording knows (all that it would keep is the empty output they write into), an autograd function is."""

    @staticmethod
    def forward(ctx, run, values, X):
        Y = X.new_empty(0)  # (an output has to be made while the recorder looks on)
        recorder = _recorder()
        torch._C._set_tracing_state(None)
        try:
            with torch.enable_grad():
                ctx.leaves = [t if t is None else t.detach().requires_grad_(need)
                              for t, need in zip((values, X), ctx.needs_input_grad[1:])]
                ctx.output = run(*ctx.leaves)
            Y.set_(ctx.output.detach())
        finally:
            torch._C._set_tracing_state(recorder)
        ctx.save_for_backward(X)  # (X overwritten, or a second backward without retain_graph: refused)
        return Y

    @staticmethod
    def backward(ctx, dY):
        ctx.saved_tensors
        wanted = [t for t, need in zip(ctx.leaves, ctx.needs_input_grad[1:]) if need]
        got = iter(torch.autograd.grad(ctx.output, wanted, dY, retain_graph=True))
        return (None, *(next(got) if need else None for need in ctx.needs_input_grad[1:]))


def spmm(graph: SparseGraph, X):
    """Differentiable Y = A X (with respect to X and, if ``graph.values`` requires grad, to the values).
    X is kept for the backward only where the values have a gradient.  Without one the backward needs nothing of the
    forward, as with torch's own linear operations: X may be overwritten before it, and it may run again without
    ``retain_graph``."""
    if _recorder() is not None:
        return _Recorded.apply(lambda values, X: _b._nat.ag_spmm(graph._native, values, X), graph.values, X)
    return _b._nat.ag_spmm(graph._native, graph.values, X)


def matmul(graph: SparseGraph, X, reduce: str = "sum"):
    """The paper's matmul(sparse, dense, reduce) (Section 3.5): reduce in 'sum' | 'mean' | 'min' | 'max'.
    Differentiable with respect to X; with respect to the edge values for 'sum' only.  min / max remember the
    position of the winning entry per output element for the backward."""
    if reduce == "sum":
        return spmm(graph, X)
    if reduce not in ("mean", "min", "max"):
        raise ValueError("reduce must be 'sum', 'mean', 'min' or 'max'")
    if graph.values is not None and graph.values.requires_grad:
        raise NotImplementedError("gradients with respect to the edge values exist for reduce='sum' only")
    if _recorder() is not None:
        return _Recorded.apply(lambda _, X: _b._nat.ag_reduce(graph._native, X, _b.REDUCE[reduce]), None, X)
    return _b._nat.ag_reduce(graph._native, X, _b.REDUCE[reduce])


def fusedmm(graph: SparseGraph, X):
    """Differentiable sigmoid FusedMM: y_i = sum_j a_ij sigmoid(<x_i, x_j>) x_j (with respect to X only)."""
    if graph.values is not None and graph.values.requires_grad:
        raise NotImplementedError("FusedMM has no gradient with respect to the edge values")
    if _recorder() is not None:
        return _Recorded.apply(lambda _, X: _b._nat.ag_fused(graph._native, X), None, X)
    return _b._nat.ag_fused(graph._native, X)
