"""SDDMM and FusedMM on both sides of the sizes at which a lane takes two vectors of a row instead of one (and SDDMM 512 columns
at a time instead of 256), at widths around what the lane shapes span, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu


def _graph(n, nnz, seed):
    rng = np.random.default_rng(seed)
    share = rng.random(n) ** 4 + 1e-3  # a few long rows
    deg = np.minimum((share / share.sum() * (nnz - n // 2)).astype(np.int64), n)
    deg[rng.permutation(n)[: n // 2]] += 1
    deg[: nnz - deg.sum()] += 1
    assert deg.sum() == nnz and deg.min() >= 0
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    rows = np.repeat(np.arange(n), deg)
    cols = rng.integers(0, n, nnz)
    cols = cols[np.lexsort((cols, rows))].astype(np.int32)
    return indptr, cols, rng.standard_normal(nnz).astype(np.float32)


@pytest.mark.parametrize("n, nnz, fused, widths", [
    (900, 6_001, True, [64, 65, 66, 128, 129, 200, 255, 256, 257, 301, 509, 512, 513, 515, 516, 602]),
    (6_000, (1 << 18) - 1, False, [65, 97, 128]), (6_000, 1 << 18, False, [65, 97, 128]),
    (9_000, (3 << 18) - 1, True, [65, 128, 257, 300, 517]), (9_000, 3 << 18, True, [65, 128, 257, 300, 517]),
    (12_000, (1 << 20) - 1, True, [129, 250]), (12_000, 1 << 20, True, [129, 250]),
    (12_288, 300_000, True, [128, 129]),  # (a directed graph's backward: one vector again beyond 6 MB)
])
def test_against_the_oracle(n, nnz, fused, widths):
    indptr, cols, values = _graph(n, nnz, n + nnz)
    A = build(indptr, cols, values)
    isp.csr_transpose_cached(A)
    rng = np.random.default_rng(2)
    for d in widths:
        print("[case] %d rows, %d entries, d = %d" % (n, nnz, d), flush=True)
        X = (0.1 * rng.standard_normal((n, d))).astype(np.float32)
        G = rng.standard_normal((n, d)).astype(np.float32)
        for scale in (False, True):
            out = torch.full((nnz,), float("nan"), device="cuda")
            isp.sddmm(A, dev(G), dev(X), out, scale_by_a=scale)
            assert_close(out, *oracle.sddmm(indptr, cols, values, G, X, scale_by_a=scale), "sddmm")
        if fused and d <= 256:
            Y = torch.full((n, d), float("nan"), device="cuda")
            isp.fusedmm(A, dev(X), Y)
            assert_close(Y, *oracle.fusedmm(indptr, cols, values, X), "fusedmm")
            Y.fill_(float("nan"))
            isp.fusedmm_backward(A, dev(X), dev(G), Y)
            assert_close(Y, *oracle.fusedmm_backward(indptr, cols, values, X, G), "fusedmm backward")
    A.destroy()


def test_one_pass_backward_on_both_sides_of_an_operand_s_size():
    """A symmetric pattern of more than 512 Ki entries, whose backward has one vector again beyond 20 MB, from 161 columns up 32 MB."""
    n = 41_000
    rng = np.random.default_rng(3)
    u, v = (n * rng.random((2, 300_000)) ** np.array([[2.0], [1.0]])).astype(np.int64)
    keys = np.unique(np.concatenate([u * n + v, v * n + u]))
    indptr = np.concatenate([[0], np.cumsum(np.bincount(keys // n, minlength=n))]).astype(np.int64)
    indices = (keys % n).astype(np.int32)
    values = rng.standard_normal(len(keys)).astype(np.float32)
    A = build(indptr, indices, values)
    isp.csr_transpose_cached(A)
    info = A.info()
    assert info["symmetric_pattern"] == 1 and 512 << 10 <= info["nnz"] < 3 << 18
    for d in (127, 128, 204, 205):
        assert (n * d <= (5 << 20 if d <= 128 else 8 << 20)) == (d in (127, 204))
        X = (0.1 * rng.standard_normal((n, d))).astype(np.float32)
        G = rng.standard_normal((n, d)).astype(np.float32)
        Y = torch.full((n, d), float("nan"), device="cuda")
        isp.fusedmm_backward(A, dev(X), dev(G), Y)
        assert_close(Y, *oracle.fusedmm_backward(indptr, indices, values, X, G), "d = %d" % d)
    A.destroy()
