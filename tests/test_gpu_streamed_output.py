"""Outputs written past the caches: one row below, at and above the size from which they are, widths that end in whole and in
partial lanes, padded and misaligned outputs whose padding stays as it was, empty rows, rows cut by runs, hub rows with and
without their fix-up launch, the mean; within tolerance of the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu

FLOATS = 16 << 20  # 64 MB


@pytest.mark.parametrize("d", [32, 37, 128, 260])
@pytest.mark.parametrize("above", [-1, 0, 1])
def test_around_the_size(d, above):
    n_rows, n_cols = -(-FLOATS // d) + above, 3_000
    rng = np.random.default_rng(d + above)
    deg = rng.integers(0, 4, n_rows)
    deg[[0, 1, n_rows // 2, n_rows - 1]] = [900, 0, 2_000, 5]  # hub rows, an empty row, a last row with entries
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    cols = rng.integers(0, n_cols, indptr[-1])
    cols = cols[np.lexsort((cols, np.repeat(np.arange(n_rows), deg)))].astype(np.int32)
    values = rng.standard_normal(len(cols)).astype(np.float32)
    X = rng.standard_normal((n_cols, d)).astype(np.float32)
    A = build(indptr, cols, values, n_cols=n_cols)
    B = isp.csr_alias(A, max_d=d)  # a fix-up launch adds its hub rows
    Xd = dev(X)
    ref, mag = oracle.spmm(indptr, cols, values, X)
    length = np.maximum(deg, 1)[:, None]
    for handle, pad, base in ((A, 0, 0), (B, 0, 0), (A, 3, 1)):
        print("[case] %d rows, d = %d, %d floats of padding, base + %d" % (n_rows, d, pad, base), flush=True)
        flat = torch.full((base + n_rows * (d + pad),), float("nan"), device="cuda")
        rows = flat[base:].view(n_rows, d + pad)
        Y = rows[:, :d]
        isp.spmm(handle, Xd, Y)
        assert_close(Y, ref, mag, "spmm")
        isp.spmm_reduce(handle, Xd, Y, "mean")
        assert_close(Y, ref / length, mag / length, "mean")
        assert torch.isnan(flat[:base]).all() and torch.isnan(rows[:, d:]).all()
    A.destroy()
