"""FusedMM two entries at a time (16, 32 and 64 lanes to a row with one vector per lane; the forward also 32 with two) and one at a time: runs that end with the first of a pair, rows that change between the two, hub segments of odd
length, and entries that a pair reads beyond its run."""
import os

import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu

N = 900


def directed(lens, seed, avoid=()):
    rng = np.random.default_rng(seed)
    cols = np.setdiff1d(np.arange(N), avoid)
    rows = [np.sort(rng.choice(cols, n, replace=False)) for n in lens]
    indptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    return indptr, np.concatenate(rows).astype(np.int32)


@pytest.fixture(params=["4", "8"], ids=["one vector", "two vectors"])
def vectors(request):
    """(Small graphs have two by themselves beyond 64 columns.)"""
    os.environ["ISP_FUSED_W"] = request.param
    yield
    os.environ.pop("ISP_FUSED_W")


# (one vector: 8, 16, 32 and 64 lanes to a row; two: 8, 16 and 32; widths that are no multiple of 4)
@pytest.mark.parametrize("d", [32, 47, 64, 65, 128, 131, 256])
@pytest.mark.parametrize("op", ["sigmoid", "dot", "one"])
def test_rows_of_every_remainder(vectors, d, op):
    rng = np.random.default_rng(d)
    lens = np.concatenate([np.arange(17).repeat(5), rng.integers(0, 12, N - 85 - 3), [701, 130, 97]])
    rng.shuffle(lens)
    indptr, indices = directed(lens, d)
    values = graphgen.uniform(indices.shape[0], 7)
    X = (0.3 * rng.standard_normal((N, d))).astype(np.float32)
    G = rng.standard_normal((N, d)).astype(np.float32)
    A = build(indptr, indices, values)
    isp.csr_transpose_cached(A)
    Y = torch.empty(N, d, device="cuda")
    isp.fusedmm(A, dev(X), Y, op=op)
    assert_close(Y, *oracle.fusedmm(indptr, indices, values, X, op=op), "forward")
    isp.fusedmm_backward(A, dev(X), dev(G), Y, op=op)
    assert_close(Y, *oracle.fusedmm_backward(indptr, indices, values, X, G, op=op), "backward")


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_values_of_rows_that_no_entry_names_stay_out(vectors, d, bad):
    rng = np.random.default_rng(d)
    lens = rng.integers(0, 10, N)
    poisoned = np.array([0, 1, 5, 450, N - 1])  # (what lies behind an item's entries reads as column 0)
    lens[poisoned] = 0
    indptr, indices = directed(lens, d, avoid=poisoned)
    X = (0.3 * rng.standard_normal((N, d))).astype(np.float32)
    X[poisoned] = bad
    A = build(indptr, indices, None)
    isp.csr_transpose_cached(A)
    Y = torch.empty(N, d, device="cuda")
    isp.fusedmm(A, dev(X), Y)
    assert bool(torch.isfinite(Y).all())
    isp.fusedmm_backward(A, dev(X), dev(np.ones((N, d), dtype=np.float32)), Y)
    assert bool(torch.isfinite(Y).all())
