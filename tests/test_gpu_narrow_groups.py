"""SpMM, SDDMM, FusedMM and min / max up to 16 columns, where four lanes hold a row: widths around it, rows of every remainder of its 16 runs, hub rows, and sizes
on both sides of those from which SpMM, FusedMM, min / max and their backward take it (the rules on the CPU: test_lane_rule.py)."""
import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu


def graph(n, nnz, seed, hubs=True):
    """Rows of 0 ... 33 entries, every length among them, and three hub rows; exactly nnz entries."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 34, n)
    lens[:34] = np.arange(34)
    if hubs:
        lens[34:37] = [900, 331, 177]
    k = n - 1
    while lens.sum() != nnz:  # (the last rows make up the difference)
        step = int(np.clip(nnz - lens.sum(), -lens[k], 60 - lens[k]))
        lens[k] += step
        k -= 1
    indptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    indices = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in lens]).astype(np.int32)
    return indptr, indices, graphgen.uniform(nnz, seed)


@pytest.mark.parametrize("d", [4, 5, 7, 8, 12, 13, 16, 17])
@pytest.mark.parametrize("nnz, hubs", [((64 << 10) - 1, True), (64 << 10, True), ((64 << 10) - 1, False), (64 << 10, False),
                                       ((96 << 10) - 1, False), (96 << 10, False), ((120 << 10) - 1, False), (120 << 10, False)])
def test_narrow_rows(d, nnz, hubs):
    n = nnz // 16
    indptr, indices, values = graph(n, nnz, d, hubs)
    rng = np.random.default_rng(d)
    X = (0.5 * rng.standard_normal((n, d))).astype(np.float32)
    G = rng.standard_normal((n, d)).astype(np.float32)
    A = build(indptr, indices, values)
    isp.csr_transpose_cached(A)
    assert (A.info()["n_hub_rows"] > 0) == hubs
    out = torch.empty(nnz, device="cuda")
    for scale in (False, True):
        isp.sddmm(A, dev(G), dev(X), out, scale_by_a=scale)
        assert_close(out, *oracle.sddmm(indptr, indices, values if scale else None, G, X, scale_by_a=scale), "sddmm")
    Y = torch.empty(n, d, device="cuda")
    for op in ("sigmoid", "dot", "one"):
        isp.fusedmm(A, dev(X), Y, op=op)
        assert_close(Y, *oracle.fusedmm(indptr, indices, values, X, op=op), "forward " + op)
        isp.fusedmm_backward(A, dev(X), dev(G), Y, op=op)
        assert_close(Y, *oracle.fusedmm_backward(indptr, indices, values, X, G, op=op), "backward " + op)


@pytest.mark.parametrize("d", [4, 6, 11, 16])
@pytest.mark.parametrize("nnz", [(512 << 10) - 1, 512 << 10])
@pytest.mark.parametrize("integers", [False, True])
def test_narrow_min_max(d, nnz, integers):
    n = 32_000
    indptr, indices, values = graph(n, nnz, d)
    rng = np.random.default_rng(d)
    X = rng.standard_normal((n, d)).astype(np.float32)
    if integers:  # many equal products: the first entry wins
        values = rng.integers(-1, 2, nnz).astype(np.float32)
        X = rng.integers(-2, 3, (n, d)).astype(np.float32)
    A = build(indptr, indices, values)
    for reduce in ("min", "max"):
        Y = torch.full((n, d), float("nan"), device="cuda")
        arg = torch.full((n, d), -7, dtype=torch.int32, device="cuda")
        isp.spmm_reduce(A, dev(X), Y, reduce, arg)
        ref, ref_arg, _ = oracle.spmm_reduce(indptr, indices, values, X, reduce)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
        assert np.array_equal(arg.cpu().numpy(), ref_arg)


@pytest.mark.parametrize("d", [4, 9, 16])
@pytest.mark.parametrize("nnz", [(768 << 10) - 1, 768 << 10])
def test_narrow_spmm(d, nnz):
    n = 48_000
    indptr, indices, values = graph(n, nnz, d)
    X = graphgen.normal((n, d), d)
    A = build(indptr, indices, values)
    Y = torch.empty(n, d, device="cuda")
    isp.spmm(A, dev(X), Y)
    assert_close(Y, *oracle.spmm(indptr, indices, values, X))


@pytest.mark.parametrize("d", [4, 11, 16, 17])
@pytest.mark.parametrize("nnz, hubs", [((256 << 10) - 1, True), ((256 << 10) - 1, False), (256 << 10, False)])
def test_narrow_max_backward(d, nnz, hubs):
    n = 16_000
    indptr, indices, values = graph(n, nnz, d, hubs)
    if hubs:  # (of the transpose, whose rows the backward takes)
        rows = np.repeat(np.arange(n), np.diff(indptr))
        indices[:: 50] = 7
        indices = indices[np.lexsort((indices, rows))]
    rng = np.random.default_rng(d)
    X = rng.integers(-2, 3, (n, d)).astype(np.float32)
    G = rng.standard_normal((n, d)).astype(np.float32)
    A = build(indptr, indices, values)
    assert (isp.csr_transpose_cached(A)[0].info()["n_hub_rows"] > 0) == hubs
    for reduce in ("min", "max"):
        Y, dX = (torch.full((n, d), float("nan"), device="cuda") for _ in range(2))
        arg = torch.full((n, d), -7, dtype=torch.int32, device="cuda")
        isp.spmm_reduce(A, dev(X), Y, reduce, arg)
        ref, ref_arg, _ = oracle.spmm_reduce(indptr, indices, values, X, reduce)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref) and np.array_equal(arg.cpu().numpy(), ref_arg)
        isp.spmm_reduce_backward(A, dev(G), dX, reduce, arg)
        assert_close(dX, *oracle.spmm_reduce_backward(n, indptr, indices, values, G, reduce, ref_arg), "backward " + reduce)


@pytest.mark.parametrize("d", [4, 7, 16])
@pytest.mark.parametrize("hubs", [False, True])
def test_narrow_one_pass_backward(d, hubs):
    """Symmetric patterns, whose FusedMM backward is one pass; the values are not symmetric."""
    n = 6_000
    rng = np.random.default_rng(d)
    u, v = rng.integers(0, n, (2, 50_000))
    if hubs:
        u[:4_000] = rng.integers(0, 5, 4_000) * 1_000
    keys = np.unique(np.concatenate([u * n + v, v * n + u]))
    assert len(keys) >= 96 << 10
    rows, indices = keys // n, (keys % n).astype(np.int32)
    indptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    values = graphgen.uniform(len(keys), d)
    X = (0.5 * rng.standard_normal((n, d))).astype(np.float32)
    G = rng.standard_normal((n, d)).astype(np.float32)
    A = build(indptr, indices, values)
    isp.csr_transpose_cached(A)
    info = A.info()
    assert info["symmetric_pattern"] == 1 and (info["n_hub_rows"] > 0) == hubs
    Y = torch.full((n, d), float("nan"), device="cuda")
    for op in ("sigmoid", "dot", "one"):
        isp.fusedmm_backward(A, dev(X), dev(G), Y, op=op)
        assert_close(Y, *oracle.fusedmm_backward(indptr, indices, values, X, G, op=op), "backward " + op)
