"""Outputs written past the caches: one row below, at and above the size from which they are, widths that end in whole and in
partial lanes, padded and misaligned outputs whose padding stays as it was, empty rows, rows cut by runs, hub rows with and
without their fix-up launch, the mean; within tolerance of the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import ABS, REL, build, dev

pytestmark = pytest.mark.gpu

FLOATS = 40 << 20  # 160 MB


def _check(d, above, n_cols):
    n_rows = -(-FLOATS // d) + above
    assert n_cols * min(d, 256) * 4 > 24 << 20  # (launches whose operand fits the L2s may run on small LDS tables, which always store ordinarily)
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
    ref, mag = (torch.from_numpy(a).cuda() for a in oracle.spmm(indptr, cols, values, X))
    length = torch.from_numpy(np.maximum(deg, 1)[:, None]).cuda()

    def close(Y, ref, mag, what):
        worst = float(((Y.double() - ref).abs() / (REL * mag + ABS)).max())
        assert worst <= 1.0, "%s: error is %.3g x the tolerance" % (what, worst)  # (NaN fails)

    for handle, pad, base in ((A, 0, 0), (B, 0, 0), (A, 3, 1)):
        print("[case] %d rows, d = %d, %d columns, %d floats of padding, base + %d" % (n_rows, d, n_cols, pad, base), flush=True)
        flat = torch.full((base + n_rows * (d + pad),), float("nan"), device="cuda")
        rows = flat[base:].view(n_rows, d + pad)
        Y = rows[:, :d]
        isp.spmm(handle, Xd, Y)
        close(Y, ref, mag, "spmm")
        isp.spmm_reduce(handle, Xd, Y, "mean")
        close(Y, ref / length, mag / length, "mean")
        assert torch.isnan(flat[:base]).all() and torch.isnan(rows[:, d:]).all()
    A.destroy()


def _columns(d):
    return (24 << 20) // (4 * min(d, 256)) + 1


@pytest.mark.parametrize("d", [32, 37, 128, 260])
@pytest.mark.parametrize("above", [-1, 0, 1])
def test_around_the_size(d, above):
    _check(d, above, _columns(d))


@pytest.mark.parametrize("d, n_cols", [(8, 0), (16, 0), (20, 0), (64, 0), (128, 82_000), (200, 0), (256, 82_000)])
def test_lane_groups(d, n_cols):
    """The other shapes of a launch: groups of 4, 8, 16 and 64 lanes, 128 whole-line columns as two slices of 64."""
    _check(d, 0, n_cols or _columns(d))
