"""The packed layout's partial rows written past the caches: one column below and at the width from which they are, at widths that end
in whole and in partial lanes; sums and means within tolerance of the oracle, and the same bits through an alias."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu

FLOATS = 22_000_000  # 88 MB of partial rows
ENV = {"ISP_HUB_THRESHOLD": "24", "ISP_SEGMENT_LEN": "16", "ISP_BLOCK_COST": "32", "ISP_MID_THRESHOLD": "8", "ISP_MIN_PIECE": "4", "ISP_BANDS": "32"}


@pytest.fixture(scope="module")
def graph():
    rng = np.random.default_rng(4)
    n, n_cols = 9_000, 3_000
    deg = rng.choice([0, 1, 7, 8, 9, 60, 300], n, p=[.05, .1, .1, .1, .1, .25, .3])
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    cols = rng.integers(0, n_cols, indptr[-1])
    cols = cols[np.lexsort((cols, np.repeat(np.arange(n), deg)))].astype(np.int32)
    values = rng.standard_normal(len(cols)).astype(np.float32)
    saved = {k: os.environ.get(k) for k in ENV}
    os.environ.update(ENV)
    try:
        A = build(indptr, cols, values, n_cols=n_cols)
    finally:
        for k, v in saved.items():
            os.environ.pop(k) if v is None else os.environ.__setitem__(k, v)
    assert FLOATS // 256 < A.info()["spmm_pieces"] < FLOATS // 132, A.info()["spmm_pieces"]
    yield n, n_cols, indptr, cols, values, A, isp.csr_alias(A, max_d=256)
    A.destroy()


@pytest.mark.parametrize("wider", [-4, -1, 0, 3, 4])
def test_around_the_size(graph, wider):
    n, n_cols, indptr, cols, values, A, B = graph
    d = -(-FLOATS // A.info()["spmm_pieces"]) + wider
    print("[case] %d pieces, d = %d" % (A.info()["spmm_pieces"], d), flush=True)
    X = np.random.default_rng(d).standard_normal((n_cols, d)).astype(np.float32)
    ref, mag = oracle.spmm(indptr, cols, values, X)
    length = np.maximum(np.diff(indptr), 1)[:, None]
    out = []
    for H in (A, B):
        Y = torch.full((n, d), float("nan"), device="cuda")
        isp.spmm(H, dev(X), Y)
        assert_close(Y, ref, mag, "spmm")
        M = torch.full((n, d), float("nan"), device="cuda")
        isp.spmm_reduce(H, dev(X), M, "mean")
        assert_close(M, ref / length, mag / length, "mean")
        out.append((Y, M))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
