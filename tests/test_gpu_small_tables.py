"""The SpMM and SDDMM kernels with small LDS tables (seven workgroups per compute unit): chosen for matrices of enough entries
whose dense operand fits the L2s.  Items as full as such tables allow (rows of the hub threshold next to a full block), rows of
every class, widths on both sides of the rule's, with and without values, sum and mean, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(900_000, False), (1_500_000, False), (1_500_000, True)])
def graph(request):
    """Rows of 0 ... hub threshold entries in no order, so that row blocks end with rows of the longest kind, and a few hubs; or
    (`many`) most entries in rows that are cut into several segments: enough work items for the rules of every width."""
    nnz, many = request.param
    rng = np.random.default_rng(nnz)
    n = 9_001
    deg = rng.choice([0, 1, 3, 30, 60, 120, 159, 160, 161, 187, 188], n, p=[.1, .1, .1, .1, .1, .1, .1, .1, .1, .05, .05])
    deg[rng.integers(0, n, 5)] = 8_000
    if many:
        deg[rng.permutation(n)[:3_900]] = 330
        deg[deg == 188] = rng.choice([0, 188], int((deg == 188).sum()))
        deg[deg < 160] //= 30
        nnz = int(deg.sum())
    deg = (deg * (nnz / deg.sum())).astype(np.int64) if deg.sum() > nnz else deg.astype(np.int64)
    deg[7] += nnz - deg.sum()
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    rows = np.repeat(np.arange(n), deg)
    cols = rng.integers(0, n, nnz)
    cols = cols[np.lexsort((cols, rows))].astype(np.int32)
    values = rng.standard_normal(nnz).astype(np.float32)
    A = build(indptr, cols, values)
    info = A.info()
    assert info["block_cost"] + info["hub_threshold"] <= 448
    assert info["n_row_blocks"] + info["n_segments"] > (15 if many else 5) * 256 * 4
    yield n, indptr, cols, values, A, build(indptr, cols, None)
    A.destroy()


@pytest.mark.parametrize("d", [4, 16, 30, 64, 65, 128, 200])
def test_against_the_oracle(graph, d):
    n, indptr, cols, values, A, U = graph
    print("[case] small tables, %d entries, d = %d" % (len(cols), d), flush=True)
    rng = np.random.default_rng(d)
    X = rng.standard_normal((n, d)).astype(np.float32)
    G = rng.standard_normal((n, d)).astype(np.float32)
    for H, v in ((A, values), (U, None)):
        Y = torch.full((n, d), float("nan"), device="cuda")
        isp.spmm(H, dev(X), Y)
        assert_close(Y, *oracle.spmm(indptr, cols, v, X), "spmm")
    Y = torch.full((n, d), float("nan"), device="cuda")
    isp.spmm_reduce(A, dev(X), Y, "mean")
    ref, mag = oracle.spmm(indptr, cols, values, X)
    length = np.maximum(np.diff(indptr), 1)[:, None]
    assert_close(Y, ref / length, mag / length, "mean")
    for scale in (False, True):
        out = torch.full((len(cols),), float("nan"), device="cuda")
        isp.sddmm(A, dev(G), dev(X), out, scale_by_a=scale)
        assert_close(out, *oracle.sddmm(indptr, cols, values, G, X, scale_by_a=scale), "sddmm")
