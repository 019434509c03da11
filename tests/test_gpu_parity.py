"""GPU parity: every entry point of the C ABI against the CPU oracle on the same seeded inputs.
Structural outputs bit-exact; floats within 1e-5 * magnitude + 1e-6 per element."""
import os

import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    print("\n[case] %s" % request.node.nodeid, flush=True)
    yield
    torch.cuda.synchronize()


def _partition_env(hub=None, seg=None, block=None, bands=None):
    for k, v in (("ISP_HUB_THRESHOLD", hub), ("ISP_SEGMENT_LEN", seg), ("ISP_BLOCK_COST", block), ("ISP_BANDS", bands)):
        if v is None:
            os.environ.pop(k, None)
        else:
            os.environ[k] = str(v)


@pytest.fixture(params=[1, 32], ids=["equal", "bands"])
def small_partition(request):
    """Small hub threshold / segment / block sizes so that tiny graphs span many work items,
    hub segments and ragged tails; hub rows in equal segments or cut at column bands."""
    _partition_env(hub=24, seg=16, block=32, bands=request.param)
    yield
    _partition_env()


def _check_transpose(A, w_indptr, w_indices, w_values, n_rows, n_cols):
    At, was = isp.csr_transpose_cached(A)
    assert not was
    At2, was2 = isp.csr_transpose_cached(A)
    assert was2 and At2 is At
    ti, tj, tv, perm = At.export()
    o_ti, o_tj, o_perm, o_tv = oracle.transpose(n_rows, n_cols, w_indptr, w_indices, w_values)
    assert np.array_equal(ti.cpu().numpy(), o_ti)
    assert np.array_equal(tj.cpu().numpy(), o_tj)
    assert np.array_equal(perm.cpu().numpy(), o_perm)
    if w_values is not None:
        assert np.array_equal(tv.cpu().numpy(), o_tv)
    else:
        assert tv is None
    return At, (o_ti, o_tj, o_tv)


def _run_all_ops(indptr, indices, values, n_rows, n_cols, d, seed, fused=True):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n_cols, d)).astype(np.float32)
    G = rng.standard_normal((n_rows, d)).astype(np.float32)
    A = build(indptr, indices, values, n_cols=n_cols)
    info = A.info()
    assert info["nnz"] == len(indices) and sum(info["bin_rows"]) == n_rows and sum(info["bin_nnz"]) == len(indices)
    deg = np.diff(indptr)
    assert info["max_degree"] == (deg.max() if n_rows else 0)
    assert info["n_hub_rows"] == int((deg > info["hub_threshold"]).sum())
    # forward
    Xd, Gd = dev(X), dev(G)
    Y = torch.full((n_rows, d), float("nan"), device="cuda")
    isp.spmm(A, Xd, Y)
    ref, mag = oracle.spmm(indptr, indices, values, X)
    assert_close(Y, ref, mag, "spmm")
    # determinism
    Y2 = torch.empty_like(Y)
    isp.spmm(A, Xd, Y2)
    assert torch.equal(Y, Y2)
    # cached transpose + backward
    At, (o_ti, o_tj, o_tv) = _check_transpose(A, indptr, indices, values, n_rows, n_cols)
    dX = torch.full((n_cols, d), float("nan"), device="cuda")
    isp.spmm(At, Gd, dX)
    ref, mag = oracle.spmm(o_ti, o_tj, o_tv, G)
    assert_close(dX, ref, mag, "spmm backward")
    # sddmm (dA) and its scaled form
    out = torch.full((len(indices),), float("nan"), device="cuda")
    isp.sddmm(A, Gd, Xd, out)
    ref, mag = oracle.sddmm(indptr, indices, values, G, X)
    assert_close(out, ref, mag, "sddmm")
    isp.sddmm(A, Gd, Xd, out, scale_by_a=True)
    ref, mag = oracle.sddmm(indptr, indices, values, G, X, scale_by_a=True)
    assert_close(out, ref, mag, "sddmm scaled")
    out2 = torch.empty_like(out)
    isp.sddmm(A, Gd, Xd, out2, scale_by_a=True)
    assert torch.equal(out, out2)  # run-to-run bitwise determinism
    if fused and n_rows == n_cols and (d <= 256 or (d <= 1024 and d % 4 == 0)):
        Xs = (0.3 * X).astype(np.float32)
        Xsd = dev(Xs)
        for op in ("sigmoid", "dot", "one"):
            Yf = torch.full((n_rows, d), float("nan"), device="cuda")
            isp.fusedmm(A, Xsd, Yf, op=op)
            ref, mag = oracle.fusedmm(indptr, indices, values, Xs, op=op)
            assert_close(Yf, ref, mag, "fusedmm " + op)
            Yf2 = torch.empty_like(Yf)
            isp.fusedmm(A, Xsd, Yf2, op=op)
            assert torch.equal(Yf, Yf2)
            dXf = torch.full((n_rows, d), float("nan"), device="cuda")
            isp.fusedmm_backward(A, Xsd, Gd, dXf, op=op)
            ref, mag = oracle.fusedmm_backward(indptr, indices, values, Xs, G, op=op)
            assert_close(dXf, ref, mag, "fusedmm backward " + op)
            dXf2 = torch.empty_like(dXf)
            isp.fusedmm_backward(A, Xsd, Gd, dXf2, op=op)
            assert torch.equal(dXf, dXf2)
    A.destroy()


@pytest.mark.parametrize("d", [1, 3, 32, 64, 100, 128, 130, 200, 256])
def test_all_ops_small_graph_many_items(small_partition, d):
    w = graphgen.make_config(1, shrink=128)  # ~1.3k nodes, power law, hubs far above the small threshold
    _run_all_ops(w.indptr, w.indices, w.values, w.n, w.n, d, seed=d)


@pytest.mark.parametrize("d", [300, 513, 1024])
def test_wide_features_tile_over_columns(small_partition, d):
    w = graphgen.make_config(1, shrink=256)
    _run_all_ops(w.indptr, w.indices, w.values, w.n, w.n, d, seed=d, fused=False)


@pytest.mark.parametrize("d", [8, 16, 30, 100, 512, 1024])
def test_sweep_widths_default_partition(d):
    """The widths of the feature-width sweep (bench.py --sweep-d) that the cases above do not cover, on the
    partition the library chooses by itself: SpMM forward and backward against the oracle, every element."""
    w = graphgen.make_config(1, shrink=8)
    rng = np.random.default_rng(d)
    X = rng.standard_normal((w.n, d)).astype(np.float32)
    A = build(w.indptr, w.indices, w.values)
    Y = torch.full((w.n, d), float("nan"), device="cuda")
    isp.spmm(A, dev(X), Y)
    assert_close(Y, *oracle.spmm(w.indptr, w.indices, w.values, X), "spmm d=%d" % d)
    At, _ = isp.csr_transpose_cached(A)
    ti, tj, _, tv = oracle.transpose(w.n, w.n, w.indptr, w.indices, w.values)
    isp.spmm(At, dev(X), Y)
    assert_close(Y, *oracle.spmm(ti, tj, tv, X), "spmm backward d=%d" % d)
    A.destroy()


@pytest.mark.parametrize("groups_per_launch", [None, 1, 2, 3])
@pytest.mark.parametrize("d", [260, 512, 516, 1024])
def test_fusedmm_wider_than_a_partial_row(small_partition, d, groups_per_launch):
    """Beyond 256 columns the score still needs whole rows while a hub segment's partial row holds 256: the
    kernels compute with whole rows and a segment stores its 256-column groups (2 at 260 and 512, the last one
    ragged at 260; 3 at 516; 4 at 1024) into as many partial rows as the scratch has room for - all of them in
    one launch by default, one, two or three per launch when capped."""
    os.environ.pop("ISP_WIDE_GROUPS", None)
    if groups_per_launch:
        os.environ["ISP_WIDE_GROUPS"] = str(groups_per_launch)
    try:
        _fusedmm_wide_case(d)
    finally:
        os.environ.pop("ISP_WIDE_GROUPS", None)


def _fusedmm_wide_case(d):
    w = graphgen.make_config(1, shrink=256)
    rng = np.random.default_rng(d)
    X = (0.1 * rng.standard_normal((w.n, d))).astype(np.float32)
    G = rng.standard_normal((w.n, d)).astype(np.float32)
    for values in (w.values, None):
        A = build(w.indptr, w.indices, values)
        assert A.info()["n_hub_rows"] > 0
        isp.csr_transpose_cached(A)
        Xd, Gd = dev(X), dev(G)
        for op in ("sigmoid", "dot", "one"):
            Y = torch.full((w.n, d), float("nan"), device="cuda")
            isp.fusedmm(A, Xd, Y, op=op)
            assert_close(Y, *oracle.fusedmm(w.indptr, w.indices, values, X, op=op), "fusedmm %s d=%d" % (op, d))
            dX = torch.full((w.n, d), float("nan"), device="cuda")
            isp.fusedmm_backward(A, Xd, Gd, dX, op=op)
            assert_close(dX, *oracle.fusedmm_backward(w.indptr, w.indices, values, X, G, op=op),
                         "fusedmm backward %s d=%d" % (op, d))
        A.destroy()


def test_one_row_owning_most_entries():
    """A single row with 150,000 entries among short ones (default partition: about two thousand segments for
    that row): the fix-ups of every kernel family combine a long chain of partial rows - SpMM and its
    backward, SDDMM, FusedMM and the reductions."""
    n, d, long_row, long_len = 3000, 64, 1500, 150_000
    rng = np.random.default_rng(77)
    lens = rng.integers(0, 9, size=n)
    lens[long_row] = long_len
    indptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    indices = np.concatenate([np.sort(rng.integers(0, n, size=k)) for k in lens]).astype(np.int32)
    values = rng.uniform(-1, 1, size=len(indices)).astype(np.float32)
    _run_all_ops(indptr, indices, values, n, n, d, seed=78)
    import test_gpu_reduce
    test_gpu_reduce._check(indptr, indices, values, n, n, d, seed=79)


def test_rectangular_unsorted_duplicates_no_values(small_partition):
    indptr, indices, values = graphgen.random_csr(700, 333, 9000, 5, sorted_cols=False, allow_dup=True)
    _run_all_ops(indptr, indices, values, 700, 333, 48, seed=1)
    _run_all_ops(indptr, indices, None, 700, 333, 128, seed=2)


def test_directed_config0_default_partition():
    w = graphgen.make_config(0)
    _run_all_ops(w.indptr, w.indices, w.values, w.n, w.n, w.d, seed=0)


def test_empty_rows_and_unit_values(small_partition):
    w = graphgen.make_config(4, shrink=256)  # directed R-MAT: about half the rows are empty
    assert (np.diff(w.indptr) == 0).sum() > w.n // 4
    _run_all_ops(w.indptr, w.indices, None, w.n, w.n, 64, seed=3)


def test_degenerate_shapes():
    # nnz = 0: outputs are zero-filled
    indptr = np.zeros(6, dtype=np.int64)
    A = build(indptr, np.zeros(0, np.int32), None, n_cols=5)
    Y = torch.full((5, 7), float("nan"), device="cuda")
    isp.spmm(A, torch.ones(5, 7, device="cuda"), Y)
    assert torch.equal(Y, torch.zeros_like(Y))
    At, _ = isp.csr_transpose_cached(A)
    ti, tj, tv, perm = At.export()
    assert torch.equal(ti, torch.zeros(6, dtype=torch.int64, device="cuda")) and tj.numel() == 0
    isp.spmm(At, torch.ones(5, 7, device="cuda"), Y)
    assert torch.equal(Y, torch.zeros_like(Y))
    # same with a 16-byte friendly width and no X at all (nothing may be read from it)
    Y8 = torch.full((5, 8), float("nan"), device="cuda")
    isp.spmm(A, torch.empty(5, 8, device="cuda"), Y8)
    assert torch.equal(Y8, torch.zeros_like(Y8))
    import ctypes
    lib = isp.load_library()
    Y8.fill_(float("nan"))
    st = lib.isp_spmm(A.handle, None, 8, 8, ctypes.c_void_p(Y8.data_ptr()), 8, None)
    torch.cuda.synchronize()
    assert st == 0 and torch.equal(Y8, torch.zeros_like(Y8))
    A.destroy()
    # n_rows = 0
    A = build(np.zeros(1, dtype=np.int64), np.zeros(0, np.int32), None, n_cols=0)
    assert A.info()["n_row_blocks"] == 0
    A.destroy()
    # 1 x 1 with a self loop
    A = build(np.array([0, 1], dtype=np.int64), np.array([0], dtype=np.int32), np.array([2.0], dtype=np.float32))
    Y = torch.empty(1, 1, device="cuda")
    isp.spmm(A, torch.full((1, 1), 3.0, device="cuda"), Y)
    assert Y.item() == 6.0
    A.destroy()


def test_leading_dimension_larger_than_d(small_partition):
    w = graphgen.make_config(1, shrink=256)
    d, ld = 96, 160
    rng = np.random.default_rng(0)
    Xfull = rng.standard_normal((w.n, ld)).astype(np.float32)
    A = build(w.indptr, w.indices, w.values)
    Xd = dev(Xfull)[:, :d]
    Ybuf = torch.full((w.n, ld), 7.0, device="cuda")
    isp.spmm(A, Xd, Ybuf[:, :d])
    ref, mag = oracle.spmm(w.indptr, w.indices, w.values, Xfull[:, :d])
    assert_close(Ybuf[:, :d].contiguous(), ref, mag, "spmm with ld > d")
    assert torch.all(Ybuf[:, d:] == 7.0), "columns beyond d were written"
    A.destroy()


def test_row_pitch_beyond_24_bits_takes_the_64_bit_gather_addresses(small_partition):
    """The grouped kernels form gather addresses with a 24-bit multiply when every byte offset fits 32 bits;
    rows 16 MiB apart (and operands of more than 4 GiB in all) must take the 64-bit variants instead."""
    n, d, ld = 288, 64, (1 << 22) + 32
    indptr, indices, values = graphgen.random_csr(n, n, 6000, seed=21)
    rng = np.random.default_rng(5)
    X = (0.3 * rng.standard_normal((n, d))).astype(np.float32)
    G = rng.standard_normal((n, d)).astype(np.float32)
    big = torch.empty((2, n, ld), device="cuda")  # 2 x 4.8 GB, only the first d columns are ever touched
    Xd, Gd = big[0, :, :d], big[1, :, :d]
    Xd.copy_(dev(X)); Gd.copy_(dev(G))
    assert Xd.stride(0) * 4 >= 1 << 24
    A = build(indptr, indices, values)
    Y = torch.full((n, d), float("nan"), device="cuda")
    isp.spmm(A, Xd, Y)
    ref, mag = oracle.spmm(indptr, indices, values, X)
    assert_close(Y, ref, mag, "spmm")
    out = torch.full((len(indices),), float("nan"), device="cuda")
    isp.sddmm(A, Gd, Xd, out, scale_by_a=True)
    ref, mag = oracle.sddmm(indptr, indices, values, G, X, scale_by_a=True)
    assert_close(out, ref, mag, "sddmm")
    isp.csr_transpose_cached(A)
    for op in ("sigmoid", "dot"):
        isp.fusedmm(A, Xd, Y, op=op)
        ref, mag = oracle.fusedmm(indptr, indices, values, X, op=op)
        assert_close(Y, ref, mag, "fusedmm " + op)
        dX = torch.full((n, d), float("nan"), device="cuda")
        isp.fusedmm_backward(A, Xd, Gd, dX, op=op)
        ref, mag = oracle.fusedmm_backward(indptr, indices, values, X, G, op=op)
        assert_close(dX, ref, mag, "fusedmm backward " + op)
    A.destroy()
    del big
    torch.cuda.empty_cache()


def test_malformed_csr_is_rejected():
    w = graphgen.make_config(0)
    bad_ptr = w.indptr.copy()
    bad_ptr[10], bad_ptr[11] = bad_ptr[11], bad_ptr[10] - 1
    with pytest.raises(isp.IspError) as e:
        build(bad_ptr, w.indices, w.values)
    assert e.value.status_name == "ISP_EBADCSR"
    bad_idx = w.indices.copy()
    bad_idx[123] = w.n
    with pytest.raises(isp.IspError) as e:
        build(w.indptr, bad_idx, w.values)
    assert e.value.status_name == "ISP_EBADCSR"
    bad_idx[123] = -1
    with pytest.raises(isp.IspError):
        build(w.indptr, bad_idx, w.values)
    A = build(w.indptr, w.indices, w.values)
    X = torch.ones(w.n, 8, device="cuda")
    with pytest.raises(isp.IspError) as e:  # backward before the transpose exists
        isp.fusedmm_backward(A, X, X, torch.empty_like(X))
    assert e.value.status_name == "ISP_EINVAL"
    for wide in (1028, 258):  # FusedMM width limits: 1024 columns; beyond 256 only multiples of 4
        with pytest.raises(isp.IspError) as e:
            isp.fusedmm(A, torch.ones(w.n, wide, device="cuda"), torch.empty(w.n, wide, device="cuda"))
        assert e.value.status_name == "ISP_EUNSUPPORTED"
    A.destroy()


def test_nonfinite_rows_do_not_leak_into_other_rows(small_partition):
    """Lanes without a live entry read row 0 of the dense operand and discard it; a NaN / Inf there
    must only reach the rows that really reference column 0."""
    w = graphgen.make_config(1, shrink=128)
    d = 64
    rng = np.random.default_rng(0)
    X = rng.standard_normal((w.n, d)).astype(np.float32)
    X[0, : d // 2] = np.nan
    X[0, d // 2:] = np.inf
    A = build(w.indptr, w.indices, w.values)
    Y = torch.empty(w.n, d, device="cuda")
    isp.spmm(A, dev(X), Y)
    touches0 = np.array([0 in w.indices[w.indptr[i]:w.indptr[i + 1]] for i in range(w.n)])
    Yh = Y.cpu().numpy()
    assert np.all(np.isfinite(Yh[~touches0])), "a non-finite value leaked into a row that does not use column 0"
    Xc = X.copy()
    Xc[0] = 0.0
    ref, mag = oracle.spmm(w.indptr, w.indices, w.values, Xc)
    assert_close(Y[torch.from_numpy(~touches0).cuda()], ref[~touches0], mag[~touches0], "rows not using column 0")
    out = torch.empty(w.nnz, device="cuda")
    G = dev(rng.standard_normal((w.n, d)).astype(np.float32))
    isp.sddmm(A, G, dev(X), out)
    uses0 = w.indices == 0
    assert np.all(np.isfinite(out.cpu().numpy()[~uses0]))
    A.destroy()


def test_two_handles_on_two_streams():
    """Different handles have separate scratch, so they may run concurrently on different streams."""
    w = graphgen.make_config(1, shrink=8)
    A1 = build(w.indptr, w.indices, w.values)
    A2 = build(w.indptr, w.indices, w.values)
    X = dev(w.X)
    Y1, Y2 = torch.empty_like(X), torch.empty_like(X)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(3):
        isp.spmm(A1, X, Y1, stream=s1)
        isp.spmm(A2, X, Y2, stream=s2)
    s1.synchronize()
    s2.synchronize()
    assert torch.equal(Y1, Y2)
    ref, mag = oracle.spmm(w.indptr, w.indices, w.values, w.X)
    assert_close(Y1, ref, mag, "spmm on a side stream")
    A1.destroy()
    A2.destroy()


@pytest.mark.parametrize("n_rows,n_cols,nnz", [(50, 1, 40), (300, 200, 5000), (1000, 3_000_000, 4096), (5000, 70_000, 16384),
                                               (4096, 4096, 4096 * 4)])
def test_transpose_shapes(n_rows, n_cols, nnz):
    """One, two and three radix passes; a single column; mostly empty columns; nnz a multiple of the sort tile."""
    indptr, indices, values = graphgen.random_csr(n_rows, n_cols, nnz, 21, sorted_cols=False, allow_dup=True)
    A = build(indptr, indices, values, n_cols=n_cols)
    _check_transpose(A, indptr, indices, values, n_rows, n_cols)
    A.destroy()


def test_trusted_build_skips_validation_only():
    w = graphgen.make_config(0)
    A = isp.csr_build(dev(w.indptr), dev(w.indices), dev(w.values), trusted=True)
    B = build(w.indptr, w.indices, w.values)
    ia, ib = A.info(), B.info()
    assert ia == ib
    X = dev(w.X)
    Ya, Yb = torch.empty_like(X), torch.empty_like(X)
    isp.spmm(A, X, Ya)
    isp.spmm(B, X, Yb)
    assert torch.equal(Ya, Yb)
    A.destroy()
    B.destroy()


@pytest.mark.parametrize("bands,min_piece", [(1, None), (2, 4), (32, 4), (32, 64), (16, None)])
@pytest.mark.parametrize("sorted_cols", [True, False])
def test_hub_rows_cut_at_column_bands(bands, min_piece, sorted_cols):
    """Hub rows are cut where their columns cross band boundaries and their segments run in order of
    first column; the cuts are binary searches that assume sorted rows.  Whatever the band settings and
    whether or not the rows are sorted (or repeat columns), every result must be the oracle's."""
    _partition_env(hub=16, seg=16, block=32)
    os.environ["ISP_BANDS"] = str(bands)
    if min_piece is not None:
        os.environ["ISP_MIN_PIECE"] = str(min_piece)
    try:
        n_rows, n_cols = 96, 700
        rng = np.random.default_rng(1000 * bands + (min_piece or 0) + int(sorted_cols))
        # a few rows far above the hub threshold (some spanning all bands, one confined to a narrow column
        # range, one hitting a single column many times), the rest short or empty
        deg = rng.integers(0, 6, size=n_rows)
        deg[[3, 40, 41, 77, 95]] = [500, 233, 17, 64, 300]
        cols = []
        for i, k in enumerate(deg):
            if i == 40:
                c = rng.integers(300, 330, size=k)        # narrow range, many repeats
            elif i == 77:
                c = np.full(k, 699)                        # one column only, the last one
            else:
                c = rng.integers(0, n_cols, size=k)        # repeats allowed
            cols.append(np.sort(c) if sorted_cols else c)
        indptr = np.zeros(n_rows + 1, dtype=np.int64)
        np.cumsum(deg, out=indptr[1:])
        indices = np.concatenate(cols).astype(np.int32)
        values = rng.standard_normal(len(indices)).astype(np.float32)
        A = build(indptr, indices, values, n_cols=n_cols)
        info = A.info()
        assert info["n_hub_rows"] == int((deg > 16).sum())
        plain = int(sum(-(-k // 16) for k in deg if k > 16))  # segments without band cuts
        assert info["n_segments"] >= plain
        if bands == 1:
            assert info["n_segments"] == plain
        if sorted_cols:  # the cut rule, restated: segments of every band piece of every hub row
            mp = min_piece if min_piece is not None else 8  # default: half the segment length
            bw = -(-n_cols // bands)
            want = 0
            for i, k in enumerate(deg):
                if k <= 16:
                    continue
                br = 1
                while br * 2 <= bands and br * 2 * mp <= k:
                    br *= 2
                step = bands // br
                cuts = [0] + [int(np.searchsorted(cols[i], j * step * bw, side="left")) for j in range(1, br)] + [int(k)]
                want += sum(-(-(b - a) // 16) for a, b in zip(cuts[:-1], cuts[1:]) if b > a)
            assert info["n_segments"] == want
        A.destroy()
        for d in (4, 32, 128):
            _run_all_ops(indptr, indices, values, n_rows, n_cols, d, seed=d, fused=False)
    finally:
        _partition_env()
        os.environ.pop("ISP_BANDS", None)
        os.environ.pop("ISP_MIN_PIECE", None)


def test_caller_owned_workspaces():
    """csr_build / csr_transpose_cached accept the caller's workspace tensors (as the C boundary does);
    a workspace below the queried size is refused; results equal those with library-side allocation."""
    w = graphgen.make_config(1, shrink=64)
    ip, ix, va = dev(w.indptr), dev(w.indices), dev(w.values)
    need = isp.csr_build_workspace(w.n, w.n, w.nnz)
    assert need > 0 and need % 256 == 0
    with pytest.raises(AssertionError):
        isp.csr_build(ip, ix, va, workspace=torch.empty(need - 256, dtype=torch.uint8, device="cuda"))
    ws_a = torch.full((need,), 0xAB, dtype=torch.uint8, device="cuda")  # stale contents must not matter
    A = isp.csr_build(ip, ix, va, workspace=ws_a)
    need_t = isp.csr_transpose_workspace(A)
    ws_t = torch.full((need_t,), 0xCD, dtype=torch.uint8, device="cuda")
    At, was = isp.csr_transpose_cached(A, workspace=ws_t)
    assert not was
    B = isp.csr_build(ip, ix, va)
    Bt, _ = isp.csr_transpose_cached(B)
    for x, y in zip(At.export(), Bt.export()):
        assert (x is None and y is None) or torch.equal(x, y)
    X = dev(w.X)
    Y1, Y2 = torch.empty_like(X), torch.empty_like(X)
    isp.spmm(A, X, Y1)
    isp.spmm(B, X, Y2)
    assert torch.equal(Y1, Y2)
    isp.spmm(At, X, Y1)
    isp.spmm(Bt, X, Y2)
    assert torch.equal(Y1, Y2)
    A.destroy()
    B.destroy()


@pytest.mark.parametrize("layout", ["ends", "one_row", "stripes", "tile_edges"])
def test_transpose_with_long_runs_of_empty_rows(layout):
    """The first sort pass rebuilds each tile's source rows from the row offsets: rows mark their first
    entry, a running maximum spreads the marks.  Long runs of empty rows put thousands of row starts on one
    position; rows that begin exactly on a sort-tile boundary (4096 entries) are the other edge."""
    rng = np.random.default_rng(7)
    n_rows, n_cols = 30_000, 900
    deg = np.zeros(n_rows, dtype=np.int64)
    if layout == "ends":          # entries only in the first and the last row
        deg[0], deg[-1] = 6000, 7000
    elif layout == "one_row":     # a single row in the middle owns every entry (several tiles)
        deg[17_123] = 20_000
    elif layout == "stripes":     # one row in a thousand is occupied
        deg[::1000] = rng.integers(1, 3000, size=len(deg[::1000]))
    else:                         # rows of exactly one tile, separated by runs of empty rows
        deg[[5, 2000, 2001, 29_999]] = 4096
    indptr = np.zeros(n_rows + 1, dtype=np.int64)
    np.cumsum(deg, out=indptr[1:])
    nnz = int(indptr[-1])
    indices = rng.integers(0, n_cols, size=nnz).astype(np.int32)
    values = rng.standard_normal(nnz).astype(np.float32)
    A = build(indptr, indices, values, n_cols=n_cols)
    _check_transpose(A, indptr, indices, values, n_rows, n_cols)
    A.destroy()
    _run_all_ops(indptr, indices, values, n_rows, n_cols, 8, seed=3, fused=False)


def test_values_changed_refreshes_the_cached_transpose(small_partition):
    """Edge values trained between epochs: the caller rewrites the values in place and tells the handle; the
    cached transpose keeps its structure, permutation and partition and carries the new values."""
    w = graphgen.make_config(1, shrink=64)
    ip, ix = dev(w.indptr), dev(w.indices)
    va = dev(w.values)
    A = isp.csr_build(ip, ix, va)
    At, _ = isp.csr_transpose_cached(A)
    G = np.random.default_rng(5).standard_normal((w.n, 24)).astype(np.float32)
    Gd, dX = dev(G), torch.empty(w.n, 24, device="cuda")
    # (the mean reduction's backward keeps value / row length per entry of the transpose: filled here with the
    # old values, it has to be filled again after the change)
    isp.spmm_reduce_backward(A, Gd, dX, "mean")
    assert_close(dX, *oracle.spmm_reduce_backward(w.n, w.indptr, w.indices, w.values, G, "mean"), "mean backward")
    new_vals = (w.values * 0.5 + 0.25).astype(np.float32)
    va.copy_(dev(new_vals))            # same tensor, new contents (e.g. a gradient step on the edge values)
    isp.csr_values_changed(A)
    At2, was = isp.csr_transpose_cached(A)
    assert was and At2 is At           # still the cached handle
    ti, tj, tv, perm = At.export()
    o_ti, o_tj, o_perm, o_tv = oracle.transpose(w.n, w.n, w.indptr, w.indices, new_vals)
    assert np.array_equal(tv.cpu().numpy(), o_tv) and np.array_equal(perm.cpu().numpy(), o_perm)
    isp.spmm(At, Gd, dX)
    assert_close(dX, *oracle.spmm(o_ti, o_tj, o_tv, G), "spmm backward after the values changed")
    Y = torch.empty(w.n, 24, device="cuda")
    isp.spmm(A, Gd, Y)
    assert_close(Y, *oracle.spmm(w.indptr, w.indices, new_vals, G), "spmm forward after the values changed")
    for _ in range(2):  # (the second call reuses what the first one filled)
        isp.spmm_reduce_backward(A, Gd, dX, "mean")
        assert_close(dX, *oracle.spmm_reduce_backward(w.n, w.indptr, w.indices, new_vals, G, "mean"),
                     "mean backward after the values changed")
    with pytest.raises(isp.IspError):
        isp.csr_values_changed(At)     # the transpose is not a source handle
    # no values / no cached transpose: accepted, nothing to do
    B = isp.csr_build(ip, ix, None)
    isp.csr_values_changed(B)
    isp.csr_transpose_cached(B)
    isp.csr_values_changed(B)
    isp.spmm_reduce_backward(B, Gd, dX, "mean")
    assert_close(dX, *oracle.spmm_reduce_backward(w.n, w.indptr, w.indices, None, G, "mean"),
                 "mean backward without stored values")
    A.destroy()
    B.destroy()


def test_c_abi_consumer_without_python():
    """The stand-alone program built next to the library uses the C ABI with the HIP runtime only (no
    Python, no PyTorch in its process) and checks SpMM, the cached-transpose backward and SDDMM itself."""
    import subprocess
    exe = os.path.join(os.path.dirname(isp.lib_path()), "abi_example")
    assert os.path.exists(exe), "abi_example is missing: run the build"
    res = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=100)
    print(res.stdout)
    assert res.returncode == 0 and res.stdout.startswith("OK"), res.stdout


@pytest.mark.parametrize("d", [4, 32, 64, 100, 128, 256])
def test_fusedmm_backward_one_pass_on_a_symmetric_pattern(small_partition, d):
    """A symmetric pattern with ascending rows makes A^T's structure equal to A's, and the backward runs as one
    pass over A with the mirrored entries' values taken from A^T.  The values here are NOT symmetric, so a
    wrong pairing of (i, j) with (j, i) shows; the two-pass form (ISP_NO_MIRROR) must agree with the oracle too,
    and a directed graph must not take the one-pass form."""
    w = graphgen.make_config(1, shrink=128)  # symmetrised R-MAT with self-loops, rows ascending
    rng = np.random.default_rng(d)
    values = rng.standard_normal(w.nnz).astype(np.float32)
    X = (0.3 * rng.standard_normal((w.n, d))).astype(np.float32)
    G = rng.standard_normal((w.n, d)).astype(np.float32)
    for mirror in (True, False):
        os.environ.pop("ISP_NO_MIRROR", None)
        if not mirror:
            os.environ["ISP_NO_MIRROR"] = "1"
        try:
            for vals in (values, None):
                A = build(w.indptr, w.indices, vals)
                assert A.info()["symmetric_pattern"] == 0  # not known before the transpose exists
                isp.csr_transpose_cached(A)
                assert A.info()["symmetric_pattern"] == 1
                for op in ("sigmoid", "dot", "one"):
                    dX = torch.full((w.n, d), float("nan"), device="cuda")
                    isp.fusedmm_backward(A, dev(X), dev(G), dX, op=op)
                    assert_close(dX, *oracle.fusedmm_backward(w.indptr, w.indices, vals, X, G, op=op),
                                 "fusedmm backward %s d=%d mirror=%s" % (op, d, mirror))
                    dX2 = torch.empty_like(dX)
                    isp.fusedmm_backward(A, dev(X), dev(G), dX2, op=op)
                    assert torch.equal(dX, dX2)
                A.destroy()
        finally:
            os.environ.pop("ISP_NO_MIRROR", None)
    w0 = graphgen.make_config(0)  # directed
    A = build(w0.indptr, w0.indices, w0.values)
    isp.csr_transpose_cached(A)
    assert A.info()["symmetric_pattern"] == 0
    A.destroy()
    # a symmetric pattern whose rows are not ascending is not recognised (and still computed correctly)
    indptr, indices = w.indptr, w.indices.copy()
    for i in range(w.n):
        s, e = indptr[i], indptr[i + 1]
        indices[s:e] = indices[s:e][::-1]
    A = build(indptr, indices, None)
    isp.csr_transpose_cached(A)
    assert A.info()["symmetric_pattern"] == (1 if np.array_equal(indices, w.indices) else 0)
    dX = torch.full((w.n, d), float("nan"), device="cuda")
    isp.fusedmm_backward(A, dev(X), dev(G), dX)
    assert_close(dX, *oracle.fusedmm_backward(indptr, indices, None, X, G), "fusedmm backward, descending rows")
    A.destroy()


@pytest.mark.parametrize("fused_w", [0, 4, 8])
@pytest.mark.parametrize("d", [36, 64, 68, 100, 128, 132, 200, 256])
def test_sddmm_and_fusedmm_lane_shapes(small_partition, d, fused_w):
    """The grouped SDDMM / FusedMM kernels give a lane one float4 or two (chosen by width and graph; ISP_FUSED_W
    forces either above 32 columns; with two the second vector is ragged or entirely past d at widths such as
    36, 68, 100, 132, 200): both shapes,
    every edge function, forward and both backward forms (directed graph: two passes; symmetric: one),
    with and without values, against the oracle element by element."""
    os.environ.pop("ISP_FUSED_W", None)
    if fused_w:
        os.environ["ISP_FUSED_W"] = str(fused_w)
    try:
        for w in (graphgen.make_config(1, shrink=128), graphgen.make_config(4, shrink=256)):
            rng = np.random.default_rng(d)
            X = (0.2 * rng.standard_normal((w.n, d))).astype(np.float32)
            G = rng.standard_normal((w.n, d)).astype(np.float32)
            for values in (w.values if w.values is not None else rng.standard_normal(w.nnz).astype(np.float32), None):
                A = build(w.indptr, w.indices, values)
                assert A.info()["n_hub_rows"] > 0
                isp.csr_transpose_cached(A)
                Xd, Gd = dev(X), dev(G)
                out = torch.full((w.nnz,), float("nan"), device="cuda")
                isp.sddmm(A, Gd, Xd, out, scale_by_a=values is not None)
                assert_close(out, *oracle.sddmm(w.indptr, w.indices, values, G, X, scale_by_a=values is not None),
                             "sddmm d=%d" % d)
                for op in ("sigmoid", "dot", "one"):
                    Y = torch.full((w.n, d), float("nan"), device="cuda")
                    isp.fusedmm(A, Xd, Y, op=op)
                    assert_close(Y, *oracle.fusedmm(w.indptr, w.indices, values, X, op=op), "fusedmm %s d=%d" % (op, d))
                    dX = torch.full((w.n, d), float("nan"), device="cuda")
                    isp.fusedmm_backward(A, Xd, Gd, dX, op=op)
                    assert_close(dX, *oracle.fusedmm_backward(w.indptr, w.indices, values, X, G, op=op),
                                 "fusedmm backward %s d=%d" % (op, d))
                    Y2, dX2 = torch.empty_like(Y), torch.empty_like(dX)
                    isp.fusedmm(A, Xd, Y2, op=op)
                    isp.fusedmm_backward(A, Xd, Gd, dX2, op=op)
                    assert torch.equal(Y, Y2) and torch.equal(dX, dX2)
                A.destroy()
    finally:
        os.environ.pop("ISP_FUSED_W", None)
