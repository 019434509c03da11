"""Widths that are no multiple of 4 and rows that start at any float: the last lane of a row moves back to end with the
last column, so it must count no column twice, read nothing beside the row and leave the columns next to it alone."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu

WIDTHS = [4, 5, 6, 7, 9, 31, 33, 62, 63, 65, 67, 127, 129, 130, 131, 158, 225, 253, 255, 257, 259, 386]


def _shifted(a, ld, off):
    """`a` as rows of a wider matrix, `off` floats in, with NaN all around."""
    buf = torch.full((a.shape[0], ld), float("nan"), device="cuda")
    v = buf[:, off:off + a.shape[1]]
    v.copy_(dev(a))
    return v, buf


def _untouched(buf, off, d):
    assert torch.isnan(buf[:, :off]).all() and torch.isnan(buf[:, off + d:]).all(), "a neighbouring column was written"


@pytest.fixture(scope="module")
def graph():
    # hub rows, empty rows, rows of one entry and rows of a few hundred
    w = graphgen.make_config(4, shrink=512)
    A = build(w.indptr, w.indices, w.values)
    At, _ = isp.csr_transpose_cached(A)
    assert A.info()["n_hub_rows"] > 0 and A.info()["bin_rows"][0] > 0
    return w, A, At


@pytest.mark.parametrize("d", WIDTHS)
def test_every_operation_at_width(graph, d):
    w, A, At = graph
    rng = np.random.default_rng(d)
    X = (0.3 * rng.standard_normal((w.n, d))).astype(np.float32)
    G = rng.standard_normal((w.n, d)).astype(np.float32)
    ld = d + 5
    Xs, _ = _shifted(X, ld, 3)
    Gs, _ = _shifted(G, ld, 1)
    print("width %d" % d, flush=True)

    Y, yb = _shifted(np.zeros_like(X), ld, 2)
    isp.spmm(A, Xs, Y)
    assert_close(Y.contiguous(), *oracle.spmm(w.indptr, w.indices, w.values, X), "spmm d=%d" % d)
    isp.spmm_reduce(A, Xs, Y, "mean")
    ref, _, mag = oracle.spmm_reduce(w.indptr, w.indices, w.values, X, "mean")
    assert_close(Y.contiguous(), ref, mag, "mean d=%d" % d)
    _untouched(yb, 2, d)

    out = torch.empty(w.nnz, device="cuda")
    isp.sddmm(A, Gs, Xs, out)
    assert_close(out, *oracle.sddmm(w.indptr, w.indices, w.values, G, X), "sddmm d=%d" % d)

    for reduce in ("min", "max"):
        arg = torch.empty(w.n, d, dtype=torch.int32, device="cuda")
        isp.spmm_reduce(A, Xs, Y, reduce, arg)
        ref, ref_arg, _ = oracle.spmm_reduce(w.indptr, w.indices, w.values, X, reduce)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref) and np.array_equal(arg.cpu().numpy(), ref_arg), reduce
        isp.spmm_reduce_backward(A, Gs, Y, reduce, arg)
        assert_close(Y.contiguous(), *oracle.spmm_reduce_backward(w.n, w.indptr, w.indices, w.values, G, reduce, ref_arg),
                     "%s backward d=%d" % (reduce, d))
        _untouched(yb, 2, d)

    if d <= 256:
        isp.fusedmm(A, Xs, Y)
        assert_close(Y.contiguous(), *oracle.fusedmm(w.indptr, w.indices, w.values, X), "fusedmm d=%d" % d)
        isp.fusedmm_backward(A, Xs, Gs, Y)
        assert_close(Y.contiguous(), *oracle.fusedmm_backward(w.indptr, w.indices, w.values, X, G), "fusedmm backward d=%d" % d)
        _untouched(yb, 2, d)
