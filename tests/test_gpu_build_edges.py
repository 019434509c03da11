"""Handle building and transposition at the sizes where their kernels change shape: row counts around a tile of rows and
around the count from which tiles grow, entry counts around a tile of keys, column counts around a digit boundary, more
hub segments than the one-launch ordering takes, and large symmetric patterns, whose transpose shares A's partitions."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu


def _random(n_rows, n_cols, nnz, seed, hub=0):
    """nnz entries in random rows, columns in no order; `hub` of them in the second row."""
    rng = np.random.default_rng(seed)
    rows = np.sort(np.concatenate([rng.integers(0, n_rows, nnz - hub), np.full(hub, min(1, n_rows - 1))]))
    indptr = np.zeros(n_rows + 1, np.int64)
    np.cumsum(np.bincount(rows, minlength=n_rows), out=indptr[1:])
    indices = rng.integers(0, n_cols, nnz).astype(np.int32)
    if hub:  # the cuts look for sorted columns
        a, b = indptr[min(1, n_rows - 1)], indptr[min(1, n_rows - 1) + 1]
        indices[a:b] = np.sort(indices[a:b])
    return indptr, indices, rng.standard_normal(nnz).astype(np.float32)


def _check(indptr, indices, values, n_cols, d=5):
    n_rows = len(indptr) - 1
    rng = np.random.default_rng(0)
    X = rng.standard_normal((n_cols, d)).astype(np.float32)
    G = rng.standard_normal((n_rows, d)).astype(np.float32)
    dv = dev(values)
    A = isp.csr_build(dev(indptr), dev(indices), dv, n_cols=n_cols)
    info, deg = A.info(), np.diff(indptr)
    assert info["max_degree"] == deg.max() and info["n_hub_rows"] == int((deg > info["hub_threshold"]).sum())
    assert sum(info["bin_rows"]) == n_rows and sum(info["bin_nnz"]) == len(indices)
    Y = torch.full((n_rows, d), float("nan"), device="cuda")
    isp.spmm(A, dev(X), Y)
    assert_close(Y, *oracle.spmm(indptr, indices, values, X), "spmm")
    At, _ = isp.csr_transpose_cached(A)
    ti, tj, tp, tv = oracle.transpose(n_rows, n_cols, indptr, indices, values)
    for got, ref in zip(At.export(), (ti, tj, tv, tp)):
        assert np.array_equal(got.cpu().numpy(), ref)
    dX = torch.full((n_cols, d), float("nan"), device="cuda")
    isp.spmm(At, dev(G), dX)
    assert_close(dX, *oracle.spmm(ti, tj, tv, G), "spmm of the transpose")
    return A, At, (ti, tj, tp), dv, G


@pytest.mark.parametrize("n_rows,n_cols,nnz,hub", [
    (1, 1, 1, 0), (1, 300, 1023, 0), (63, 255, 1024, 0), (64, 256, 1025, 0), (65, 257, 4097, 2500),
    (255, 511, 5000, 0), (256, 512, 5000, 4000), (257, 513, 5000, 0), (700, 65537, 30000, 20000),
    (100, 131072, 9000, 0), (100, 131073, 9000, 0), (3, 262145, 9000, 5000),
    (262143, 50, 60000, 9000), (262144, 50, 60000, 9000), (262145, 50, 60000, 9000), (1048577, 50, 60000, 9000),
    (3000, 1000, (4 << 20), 70000), (3000, 1000, (4 << 20) + 1, 70000)])
def test_tile_edges(n_rows, n_cols, nnz, hub):
    print("rows %d cols %d nnz %d" % (n_rows, n_cols, nnz), flush=True)
    _check(*_random(n_rows, n_cols, nnz, n_rows + nnz, hub), n_cols)


@pytest.mark.parametrize("n_rows,n_cols,nnz", [(64, 256, 1025), (65, 257, 4097), (100, 131073, 9000), (3000, 1 << 20, 50000),
                                               (5, 1 << 26, 3000)])
def test_pattern_only_transposes(n_rows, n_cols, nnz):
    """One to four passes of the sort without values (records of a small matrix still hold four numbers)."""
    print("rows %d cols %d nnz %d, no values" % (n_rows, n_cols, nnz), flush=True)
    indptr, indices, _ = _random(n_rows, n_cols, nnz, nnz)
    At, _ = isp.csr_transpose_cached(build(indptr, indices, None, n_cols=n_cols))
    ti, tj, tp, _ = oracle.transpose(n_rows, n_cols, indptr, indices, None)
    got = At.export()
    assert got[2] is None
    for g, ref in ((got[0], ti), (got[1], tj), (got[3], tp)):
        assert np.array_equal(g.cpu().numpy(), ref)


@pytest.mark.parametrize("at", [0, 4_999_999])
def test_column_out_of_range_is_reported(at):
    """Few rows, many entries: the workgroup that meets the bad column need not own any rows."""
    print("bad column at %d" % at, flush=True)
    indices = np.zeros(5_000_000, np.int32)
    indices[at] = 7
    with pytest.raises(isp.IspError) as e:
        build(np.array([0, 1_000_000, 2_000_000, 5_000_000], np.int64), indices, None, n_cols=7)
    assert e.value.status_name == "ISP_EBADCSR"


def test_overlapping_rows_are_reported():
    """Every second row claims all entries: more segments together than 32 bits count."""
    n_rows, nnz = 600_000, 1_000_000
    print("overlapping rows", flush=True)
    indptr = np.zeros(n_rows + 1, np.int64)
    indptr[1::2] = nnz
    indptr[-1] = nnz
    assert n_rows // 2 * (nnz // ((n_rows + nnz) // 16384)) > 1 << 31  # (segments of a quarter of a wavefront slot's share)
    for trusted in (False, True):
        with pytest.raises(isp.IspError) as e:
            isp.csr_build(dev(indptr), torch.zeros(nnz, dtype=torch.int32, device="cuda"), None, n_cols=50, trusted=trusted)
        assert e.value.status_name == "ISP_EBADCSR"


@pytest.mark.parametrize("n_hub", [8191, 8192, 8193, 20000])
def test_many_segments(n_hub):
    print("hub rows %d" % n_hub, flush=True)
    os.environ["ISP_HUB_THRESHOLD"] = "16"
    try:
        rng = np.random.default_rng(n_hub)
        deg = np.concatenate([np.full(n_hub, 17), rng.integers(0, 9, 1000)])
        rng.shuffle(deg)
        indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
        indices = rng.integers(0, 4000, indptr[-1]).astype(np.int32)
        A, *_ = _check(indptr, indices, rng.standard_normal(indptr[-1]).astype(np.float32), 4000)
        assert A.info()["n_segments"] >= n_hub
    finally:
        os.environ.pop("ISP_HUB_THRESHOLD")


@pytest.mark.parametrize("n_hub", [12345, 16384, 16385])
def test_segments_beyond_one_table(n_hub):
    """More keys than the ranking holds at a time, as many as it takes, and one more: the radix sort."""
    test_many_segments(n_hub)


@pytest.mark.parametrize("mid,with_values", [(0, True), (64, True), (64, False)])
def test_large_symmetric(mid, with_values):
    print("threshold %d" % mid, flush=True)
    os.environ["ISP_MID_THRESHOLD"] = str(mid)
    try:
        rng = np.random.default_rng(7)
        n = 70000
        i, j = rng.integers(0, n, 2300000), rng.integers(0, n, 2300000)
        i[:40000] = 5  # a hub
        code = np.unique(np.concatenate([i * n + j, j * n + i]))
        indptr = np.concatenate([[0], np.cumsum(np.bincount(code // n, minlength=n))]).astype(np.int64)
        indices = (code % n).astype(np.int32)
        assert len(indices) > 4 << 20
        values = rng.standard_normal(len(indices)).astype(np.float32) if with_values else None
        if with_values:
            A, At, (ti, tj, tp), dv, G = _check(indptr, indices, values, n)
            # rewritten values reach the transpose and both packed layouts
            new = torch.randn(len(indices), device="cuda")
            dv.copy_(new)
            isp.csr_values_changed(A)
            dX = torch.empty(n, 5, device="cuda")
            isp.spmm(At, dev(G), dX)
            assert_close(dX, *oracle.spmm(ti, tj, new.cpu().numpy()[tp], G), "after new values")
            isp.spmm(A, dev(G), dX)
            assert_close(dX, *oracle.spmm(indptr, indices, new.cpu().numpy(), G), "the matrix itself, after new values")
        else:
            A = build(indptr, indices, None)
            At, _ = isp.csr_transpose_cached(A)
            G = rng.standard_normal((n, 5)).astype(np.float32)
            dX = torch.empty(n, 5, device="cuda")
            isp.spmm(At, dev(G), dX)
            assert_close(dX, *oracle.spmm(indptr, indices, None, G), "without values")
        assert A.info()["symmetric_pattern"] == 1 and (A.info()["spmm_pieces"] > 0) == (mid > 0)
        assert At.info()["spmm_pieces"] == A.info()["spmm_pieces"] and At.info()["is_transpose"] == 1
        # both handles at once, each on a stream of its own, as when they kept separate tables
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        Xd = torch.randn(n, 64, device="cuda")
        Y1, Y2, ref1, ref2 = (torch.empty(n, 64, device="cuda") for _ in range(4))
        isp.spmm(A, Xd, ref1)
        isp.spmm(At, Xd, ref2)
        torch.cuda.synchronize()
        for _ in range(3):
            isp.spmm(A, Xd, Y1, stream=s1)
            isp.spmm(At, Xd, Y2, stream=s2)
        torch.cuda.synchronize()
        assert torch.equal(Y1, ref1) and torch.equal(Y2, ref2)
    finally:
        os.environ.pop("ISP_MID_THRESHOLD")


def test_large_symmetric_with_more_pieces_than_segment_rows():
    """Rows of about 290 entries: the packed layout cuts each into four pieces, more partial rows than the ordinary partition
    is laid out for.  The shared transpose's scratch holds them in front of its packed values, which stay as they are."""
    n, half = 70000, 145 * 70000
    g = torch.Generator(device="cuda").manual_seed(3)
    i, j = (torch.randint(n, (half,), device="cuda", generator=g) for _ in range(2))
    code = torch.unique(torch.cat([i * n + j, j * n + i]))
    indptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(code // n, minlength=n), 0, out=indptr[1:])
    indices = (code % n).to(torch.int32)
    values = torch.randn(len(code), device="cuda", generator=g)
    A = isp.csr_build(indptr, indices, values)
    info = A.info()
    seg, hub = info["segment_len"], info["hub_threshold"]
    laid_out = info["nnz"] // seg + info["nnz"] // 128 + info["nnz"] // (hub + 1) + 2
    assert info["spmm_pieces"] > laid_out, info  # (what this test is about)
    At, _ = isp.csr_transpose_cached(A)
    assert At.info()["symmetric_pattern"] == 1 and At.info()["spmm_pieces"] == info["spmm_pieces"]
    B = isp.csr_alias(A, 128)
    h_indptr, h_indices = indptr.cpu().numpy(), indices.cpu().numpy()
    X = np.random.default_rng(0).standard_normal((n, 5)).astype(np.float32)

    def check(handle, what):
        ti, tj, _, tv = oracle.transpose(n, n, h_indptr, h_indices, values.cpu().numpy())
        ref, mag = oracle.spmm(ti, tj, tv, X)
        for k in range(2):  # the second call reads the packed values that the first one's partial rows lie in front of
            Y = torch.full((n, 5), float("nan"), device="cuda")
            isp.spmm(handle, dev(X), Y)
            assert_close(Y, ref, mag, "%s, call %d" % (what, k))

    check(At, "transpose")
    check(B._At, "alias of the transpose")
    values.copy_(torch.randn(len(code), device="cuda", generator=g))
    isp.csr_values_changed(A)
    check(At, "transpose, new values")
    Y = torch.empty(n, 5, device="cuda")
    isp.spmm(A, dev(X), Y)
    assert_close(Y, *oracle.spmm(h_indptr, h_indices, values.cpu().numpy(), X), "the matrix itself")


@pytest.mark.parametrize("n_rows,n_cols", [(20000, 70001), (300000, 1000), (16385, 63), (3, 9)])
def test_rewritten_values_of_long_columns(n_rows, n_cols):
    """The transpose's values gathered block of rows by block of rows: long, short and empty parts, columns past the last."""
    print("rows %d cols %d" % (n_rows, n_cols), flush=True)
    nnz = (16 << 20) + 5
    g = torch.Generator(device="cuda").manual_seed(n_cols)
    rows = torch.randint(n_rows, (nnz,), device="cuda", generator=g)
    cols = (torch.rand(nnz, device="cuda", generator=g) ** 3 * n_cols).to(torch.int32)  # the first columns are long
    indptr = torch.zeros(n_rows + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(rows, minlength=n_rows), 0, out=indptr[1:])
    values = torch.ones(nnz, device="cuda")
    A = isp.csr_build(indptr, cols, values, n_cols=n_cols)
    At, _ = isp.csr_transpose_cached(A)
    values.copy_(torch.randn(nnz, device="cuda", generator=g))
    isp.csr_values_changed(A)
    _, _, t_values, perm = At.export()
    assert torch.equal(t_values, values[perm.long()])


def test_rewritten_values_of_more_blocks_than_a_grid_dimension_holds():
    """1.07 G rows, most of them empty: 65,552 blocks of rows."""
    n_rows, n_cols, nnz = 1_074_000_000, 60, (16 << 20) + 5
    g = torch.Generator(device="cuda").manual_seed(1)
    rows = torch.randint(n_rows, (nnz,), device="cuda", generator=g)
    rows[:8] = n_rows - 1
    cols = torch.randint(n_cols, (nnz,), device="cuda", generator=g, dtype=torch.int32)
    indptr = torch.zeros(n_rows + 1, dtype=torch.int64, device="cuda")
    indptr[1:].scatter_add_(0, rows, torch.ones_like(rows))
    torch.cumsum(indptr, 0, out=indptr)
    values = torch.ones(nnz, device="cuda")
    A = isp.csr_build(indptr, cols, values, n_cols=n_cols)
    At, _ = isp.csr_transpose_cached(A)
    for _ in range(2):  # the bounds are found by the first call and kept
        values.copy_(torch.randn(nnz, device="cuda", generator=g))
        isp.csr_values_changed(A)
        _, _, t_values, perm = At.export()
        assert torch.equal(t_values, values[perm.long()])
    A.destroy()


@pytest.mark.parametrize("n_rows", [500, 262_145, 1_100_000])
@pytest.mark.parametrize("lengths", [[4], [0, 4, 5, 32, 33, 64, 65, 200]])
def test_row_classes(n_rows, lengths):
    """Rows and entries per degree class and the longest row, exactly: rows of one length, and of lengths around every class's edge, in
    tiles of one step and of several."""
    print("%d rows" % n_rows, flush=True)
    rng = np.random.default_rng(n_rows)
    deg = rng.choice(lengths, n_rows, p=None if len(lengths) == 1 else [.3, .3, .2, .1, .04, .03, .02, .01])
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    A = build(indptr, rng.integers(0, 1000, indptr[-1]).astype(np.int32), None, n_cols=1000)
    info = A.info()
    bins = np.digitize(deg, [1, 5, 33, info["hub_threshold"] + 1])
    assert list(info["bin_rows"]) == [int((bins == k).sum()) for k in range(5)]
    assert list(info["bin_nnz"]) == [int(deg[bins == k].sum()) for k in range(5)]
    assert info["max_degree"] == deg.max() and info["n_hub_rows"] == int((bins == 4).sum())
    A.destroy()
