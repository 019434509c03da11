"""Partitions on both sides of the sizes where their rules change: the longest row of a block, the segments' length, and whether
hub rows are cut at column bands or into equal segments.  Rows of a block's longest kind, one entry more, whole segments and one
entry more, and a row of hundreds of segments (more than lanes), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu

SLOTS = 4096  # wavefront slots of the device


def _graph(n, n_cols, nnz, hub, seg):
    rng = np.random.default_rng(n + nnz)
    special = [hub, hub + 1, 2 * seg, 2 * seg + 1, 3 * seg, hub - 1, 65 * seg + 1, 0]
    deg = np.zeros(n, np.int64)
    rest = nnz - sum(special)
    deg[len(special):] = rest // (n - len(special))
    deg[len(special):][: rest % (n - len(special))] += 1
    deg[: len(special)] = special
    deg = rng.permutation(deg)
    assert deg.sum() == nnz and deg.min() >= 0
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    rows = np.repeat(np.arange(n), deg)
    cols = rng.integers(0, n_cols, nnz)
    cols = cols[np.lexsort((cols, rows))].astype(np.int32)
    return indptr, cols, rng.standard_normal(nnz).astype(np.float32)


@pytest.mark.parametrize("share, more, n, n_cols, hub, seg, banded", [
    (28, 0, 2_000, 2_000, 64, 48, False), (28, 1, 2_000, 2_000, 96, 64, False),
    (128, 0, 9_000, 9_000, 96, 64, False), (128, 1, 9_000, 9_000, 160, 80, False),
    (320, 0, 70_000, 70_000, 160, 80, False), (320, 1, 70_000, 70_000, 160, 80, True), (320, 1, 30_000, 65_535, 160, 80, False),
    (1024, 0, 65_535, 65_535, 512, 256, False), (1024, 1, 65_535, 65_535, 512, 256, True), (400, 0, 60_000, 65_535, 200, 100, False), (400, 0, 60_000, 65_536, 200, 100, True),
])
def test_both_sides_of_a_size(share, more, n, n_cols, hub, seg, banded):
    nnz = share * SLOTS + more - n
    print("[case] %d + %d units, %d rows" % (share, more, n), flush=True)
    indptr, cols, values = _graph(n, n_cols, nnz, hub, seg)
    A = build(indptr, cols, values, n_cols=n_cols)
    info = A.info()
    assert (info["hub_threshold"], info["segment_len"]) == (hub, seg)
    deg = np.diff(indptr)
    equal = int((-(-deg[deg > hub] // seg)).sum())  # (a row that is cut at bands has segments that end there as well)
    assert info["n_segments"] > equal if banded else info["n_segments"] == equal
    rng = np.random.default_rng(1)
    for d in (20, 136):
        X = (0.1 * rng.standard_normal((n_cols, d))).astype(np.float32)
        G = rng.standard_normal((n, d)).astype(np.float32)
        Y = torch.full((n, d), float("nan"), device="cuda")
        isp.spmm(A, dev(X), Y)
        assert_close(Y, *oracle.spmm(indptr, cols, values, X), "spmm")
        out = torch.full((nnz,), float("nan"), device="cuda")
        isp.sddmm(A, dev(G), dev(X), out)
        assert_close(out, *oracle.sddmm(indptr, cols, values, G, X), "sddmm")
        if n == n_cols and share <= 320:
            Y.fill_(float("nan"))
            isp.fusedmm(A, dev(X), Y)
            assert_close(Y, *oracle.fusedmm(indptr, cols, values, X), "fusedmm")
    ti, tj, perm, tv = oracle.transpose(n, n_cols, indptr, cols, values)
    At = isp.csr_transpose_cached(A)[0]
    g_ti, g_tj, g_tv, g_perm = At.export()
    assert np.array_equal(g_ti.cpu().numpy(), ti) and np.array_equal(g_tj.cpu().numpy(), tj)
    assert np.array_equal(g_perm.cpu().numpy(), perm) and np.array_equal(g_tv.cpu().numpy(), tv)
    dX = torch.full((n_cols, 20), float("nan"), device="cuda")
    dY = rng.standard_normal((n, 20)).astype(np.float32)
    isp.spmm(At, dev(dY), dX)
    assert_close(dX, *oracle.spmm(ti, tj, tv, dY), "spmm backward")
    A.destroy()
