"""SDDMM's sums of four steps at a time: runs of every length modulo four (items of few entries, so that lane groups have runs of
0, 1, 2, ... entries), every lane shape, widths that are no multiple of 4, scaled and not, added up over column windows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu


def _check(lengths, n_cols, widths, seed):
    rng = np.random.default_rng(seed)
    indptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    nnz, n = int(indptr[-1]), len(lengths)
    cols = rng.integers(0, n_cols, nnz).astype(np.int32)
    values = rng.standard_normal(nnz).astype(np.float32)
    A = build(indptr, cols, values, n_cols=n_cols)
    for d in widths:
        print("[case] sddmm, %d entries, d = %d" % (nnz, d), flush=True)
        U = rng.standard_normal((n, d)).astype(np.float32)
        V = rng.standard_normal((n_cols, d)).astype(np.float32)
        for scale in (False, True):
            out = torch.full((nnz,), float("nan"), device="cuda")
            isp.sddmm(A, dev(U), dev(V), out, scale_by_a=scale)
            assert_close(out, *oracle.sddmm(indptr, cols, values, U, V, scale_by_a=scale), "sddmm d=%d" % d)
    A.destroy()


@pytest.mark.parametrize("total", [1, 2, 3, 5, 7, 8, 13, 31, 64, 200])
def test_short_runs(total):
    """`total` entries in rows of 0 to 3: with up to 16 cost units to an item, groups get runs of 0 to 4 entries."""
    rng = np.random.default_rng(total)
    lengths = rng.integers(0, 4, 4 * total)
    lengths = lengths[np.cumsum(lengths) <= total]
    lengths = np.append(lengths, [total - lengths.sum()])
    _check(lengths, 37, [4, 6, 32, 33, 64, 65, 100, 128, 130, 192, 256, 260], total)


def test_one_group_to_a_wavefront():
    """More than 192 columns on more than a million entries: 64 lanes to an entry; the columns beyond 256 in a second pass."""
    lengths = np.random.default_rng(3).choice([0, 1, 2, 5, 90, 400], 13_000)
    lengths[0] += max(0, (1 << 20) + 3 - int(lengths.sum()))
    _check(lengths, 500, [193, 250, 256, 300], 4)
