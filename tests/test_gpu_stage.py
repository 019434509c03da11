"""Ragged dense operands of SpMM copied to whole lines (rows that start between 128-byte lines, many entries per column):
forced onto small graphs, at widths around the copies' tiles, at pitches and base addresses of every alignment, against the
oracle; bit-identical through an alias and the static-scratch entry point, also where those gather from the operand itself;
on the packed layout, in the mean and its backward, after rewritten values and in a captured graph."""
import os

import numpy as np
import pytest
import torch

import graphgen
import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    os.environ["ISP_STAGE_MIN"] = "1"
    try:
        w = graphgen.make_config(1, shrink=64)
        A = build(w.indptr, w.indices, w.values)
        At, _ = isp.csr_transpose_cached(A)
    finally:
        os.environ.pop("ISP_STAGE_MIN")
    yield w, A, At, oracle.transpose(w.n, w.n, w.indptr, w.indices, w.values)
    A.destroy()


def _operand(rng, n, d, ld, shift):
    """(n, d) view with rows ld apart that starts `shift` floats behind a line; NaN everywhere else."""
    buf = torch.full((n * ld + shift + 32,), float("nan"), device="cuda")
    V = buf[shift:shift + n * ld].view(n, ld)[:, :d]
    Xh = rng.standard_normal((n, d)).astype(np.float32)
    V.copy_(torch.from_numpy(Xh))
    return V, Xh


# widths: below / at / above one copied tile, a last tile narrower than a float4 lane, several tiles; pitches: the width
# itself, padded, whole lines (with a shifted base)
@pytest.mark.parametrize("d,ld,shift", [(4, 4, 0), (5, 5, 1), (31, 31, 0), (33, 40, 0), (64, 64, 3), (127, 127, 0), (128, 128, 1),
                                        (129, 129, 0), (131, 132, 2), (200, 200, 0), (259, 301, 5), (602, 602, 0)])
def test_against_the_oracle(graph, d, ld, shift):
    w, A, At, (ti, tj, _, tv) = graph
    print("[case] staged", d, ld, shift, flush=True)
    rng = np.random.default_rng(d)
    X, Xh = _operand(rng, w.n, d, ld, shift)
    Y = torch.full((w.n, d), float("nan"), device="cuda")
    isp.spmm(A, X, Y)
    assert_close(Y, *oracle.spmm(w.indptr, w.indices, w.values, Xh), "staged spmm")
    again = torch.empty_like(Y)
    isp.spmm_static_scratch(A, X, again)  # (the same launches, copies of its own or none)
    assert torch.equal(Y, again)
    B = isp.csr_alias(A, max_d=d)
    isp.spmm(B, X, again)
    assert torch.equal(Y, again)
    isp.spmm(At, X, Y)
    assert_close(Y, *oracle.spmm(ti, tj, tv, Xh), "staged spmm on the transpose")
    isp.spmm(isp.csr_transpose_cached(B)[0], X, again)
    assert torch.equal(Y, again)
    B.destroy()


def _graph_with_hubs(n, per_row, seed=0):
    rng = np.random.default_rng(seed)
    rows = np.concatenate([rng.integers(0, n, n * per_row), np.repeat([7, 8, n - 1], 700)])
    code = np.unique(rows * n + rng.integers(0, n, rows.size))
    indptr = np.concatenate([[0], np.cumsum(np.bincount(code // n, minlength=n))]).astype(np.int64)
    return indptr, (code % n).astype(np.int32), rng.standard_normal(code.size).astype(np.float32)


# The copies' place in the workspace: among the packed layout's idle partial rows (many entries per column), in place of
# the ordinary partition's (few: the copies then need all of them), behind it (no packed layout).
@pytest.mark.parametrize("per_row,mid", [(60, 16), (5, 100), (60, 0)])
@pytest.mark.parametrize("d", [20, 130, 301])
def test_places_of_the_copies(per_row, mid, d):
    print("[case] place", per_row, mid, d, flush=True)
    n, rng = 3000, np.random.default_rng(per_row)
    indptr, indices, values = _graph_with_hubs(n, per_row)
    env = {"ISP_STAGE_MIN": "1", "ISP_MID_THRESHOLD": str(mid)}
    os.environ.update(env)
    try:
        A = build(indptr, indices, values)
        At, _ = isp.csr_transpose_cached(A)
    finally:
        for k in env:
            os.environ.pop(k)
    assert (A.info()["spmm_pieces"] > 0) == (mid > 0) and A.info()["n_segments"] > 0
    X, Xh = _operand(rng, n, d, d, 1)
    Y, Z, dX = (torch.full((n, d), float("nan"), device="cuda") for _ in range(3))
    arg = torch.empty(n, d, dtype=torch.int32, device="cuda")
    ref = oracle.spmm(indptr, indices, values, Xh)
    ti, tj, _, tv = oracle.transpose(n, n, indptr, indices, values)
    for _ in range(2):  # (and among the partial rows of other operations: the calls on a handle follow each other)
        isp.spmm(A, X, Y)
        assert_close(Y, *ref, "spmm")
        isp.spmm_reduce(A, X, Z, "max", arg)
        top, at, _ = oracle.spmm_reduce(indptr, indices, values, Xh, "max")
        assert np.array_equal(Z.cpu().numpy(), top) and np.array_equal(arg.cpu().numpy(), at)
        isp.spmm(At, X, dX)
        assert_close(dX, *oracle.spmm(ti, tj, tv, Xh), "spmm on the transpose")
        isp.fusedmm(A, X[:, :20], Z[:, :20])
        assert_close(Z[:, :20], *oracle.fusedmm(indptr, indices, values, np.ascontiguousarray(Xh[:, :20])), "fusedmm")
    # an alias for narrow calls has little room or none; wider ones still give the same bits
    for max_d in (3, 16, d):
        B = isp.csr_alias(A, max_d=max_d)
        isp.spmm(B, X, Z)
        assert torch.equal(Y, Z)
        isp.spmm(isp.csr_transpose_cached(B)[0], X, Z)
        assert torch.equal(dX, Z)
        B.destroy()
    assert isp.csr_alias_workspace(A, max_d=128) - isp.csr_alias_workspace(A, max_d=16) == 2 * 4 * n * (128 - 16)
    assert isp.csr_alias_workspace(A, max_d=16) - isp.csr_alias_workspace(A, max_d=3) == 2 * 4 * n * 16
    A.destroy()


# 602: four tiles of 128 and one of 90; 131: a tile of 128, then one of four columns that starts before it ends, whose copy
# has rows of 8 floats, and with it a second pitch in the same scratch
@pytest.mark.parametrize("d", [20, 131, 602])
@pytest.mark.parametrize("mid", [16, 0])
def test_reductions_new_values_and_replays(mid, d):
    print("[case] staged mean, new values, graph", mid, d, flush=True)
    n, rng = 2000, np.random.default_rng(d)
    indptr, indices, values = _graph_with_hubs(n, 40)
    env = {"ISP_STAGE_MIN": "1", "ISP_MID_THRESHOLD": str(mid)}
    os.environ.update(env)
    try:
        vals = torch.from_numpy(values.copy()).cuda()
        A = isp.csr_build(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), vals)
        At, _ = isp.csr_transpose_cached(A)
    finally:
        for k in env:
            os.environ.pop(k)
    assert (A.info()["spmm_pieces"] > 0) == (mid > 0)
    X, Xh = _operand(rng, n, d, d, 1)
    G, Gh = _operand(rng, n, d, d + 2, 0)
    Y, M, dX, dM = outs = [torch.full((n, d), float("nan"), device="cuda") for _ in range(4)]

    def step():
        isp.spmm(A, X, Y)
        isp.spmm_reduce(A, X, M, "mean")
        isp.spmm(At, G, dX)
        isp.spmm_reduce_backward(A, G, dM, "mean")

    def check(values, what):
        ti, tj, _, tv = oracle.transpose(n, n, indptr, indices, values)
        assert_close(Y, *oracle.spmm(indptr, indices, values, Xh), what + ", spmm")
        assert_close(dX, *oracle.spmm(ti, tj, tv, Gh), what + ", spmm of the transpose")
        ref, _, mag = oracle.spmm_reduce(indptr, indices, values, Xh, "mean")
        assert_close(M, ref, mag, what + ", mean")
        assert_close(dM, *oracle.spmm_reduce_backward(n, indptr, indices, values, Gh, "mean"), what + ", mean backward")

    step()
    check(values, "eager")
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        step()
    torch.cuda.synchronize()
    for rep in range(3):  # every replay on new values and new operands, with eager work of the handle before it
        new = rng.standard_normal(values.size).astype(np.float32)
        vals.copy_(torch.from_numpy(new))
        isp.csr_values_changed(A)
        isp.spmm(A, torch.randn(n, 37, device="cuda"), torch.empty(n, 37, device="cuda"))
        Xh[:] = rng.standard_normal((n, d))
        X.copy_(torch.from_numpy(Xh))
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check(new, "replay %d" % rep)
    A.destroy()


def _holds_copy(ws, X, c0, pitch):
    """Do the rows of the columns [c0, ...) of X, up to the last one, lie `pitch` floats apart somewhere in the workspace ws?"""
    part = X[:, c0:]
    n, w = part.shape
    mem = ws[: ws.numel() // 4 * 4].view(torch.float32)
    for at in torch.nonzero(mem == part[0, 0]).flatten().tolist():
        if at + n * pitch <= mem.numel() and torch.equal(mem[at:at + n * pitch].view(n, pitch)[:, :w], part):
            return True
    return False


def _build_in(ws_of, indptr, indices, values, **env):
    """(A, its transpose, their workspaces) with the environment `env` set meanwhile."""
    os.environ.update(env)
    try:
        n = len(indptr) - 1
        ws = ws_of(isp.csr_build_workspace(n, n, len(indices)))
        A = isp.csr_build(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), torch.from_numpy(values).cuda(), workspace=ws)
        wst = ws_of(isp.csr_transpose_workspace(A))
        At, _ = isp.csr_transpose_cached(A, workspace=wst)
    finally:
        for k in env:
            os.environ.pop(k)
    return A, At, ws, wst


def _clean(nbytes):
    return torch.zeros(nbytes, dtype=torch.uint8, device="cuda")


# (131 columns: the last tile's copy has rows of 8 floats)
@pytest.mark.parametrize("d,c0,pitch", [(7, 0, 8), (20, 0, 32), (100, 0, 128), (131, 127, 8), (300, 256, 64)])
@pytest.mark.parametrize("mid", [16, 0])
def test_copies_are_made(mid, d, c0, pitch):
    """The handle's workspace holds the last tile's columns after a call, and a call without copies leaves none there."""
    print("[case] copies made", mid, d, flush=True)
    g = _graph_with_hubs(2500, 30)
    A, At, ws, wst = _build_in(_clean, *g, ISP_STAGE_MIN="1", ISP_MID_THRESHOLD=str(mid))
    for h, mem in ((A, ws), (At, wst)):
        X = torch.randn(2500, d, device="cuda")
        isp.spmm(h, X, torch.empty_like(X))
        assert _holds_copy(mem, X, c0, pitch)
        X = torch.randn(2500, 128, device="cuda")  # (whole lines)
        isp.spmm(h, X, torch.empty_like(X))
        assert not _holds_copy(mem, X, 0, 128)
    B = isp.csr_alias(A, max_d=d, workspace=(wsb := _clean(isp.csr_alias_workspace(A, max_d=d))))
    X = torch.randn(2500, d, device="cuda")
    isp.spmm(B, X, torch.empty_like(X))
    assert _holds_copy(wsb, X, c0, pitch) and not _holds_copy(ws, X, c0, pitch)
    X = torch.randn(2500, d, device="cuda")
    isp.spmm_static_scratch(A, X, torch.empty_like(X))
    assert _holds_copy(ws, X, c0, pitch)
    B.destroy()
    A.destroy()


# from 80 Ki columns (512 Ki on the packed layout) a tile of 128 copied columns is gathered as two slices of 64
@pytest.mark.parametrize("n,per_row,mid", [(90_001, 12, 0), (524_301, 5, 16)])
@pytest.mark.parametrize("d,c0,pitch", [(131, 127, 8), (150, 128, 32)])
def test_copies_in_two_slices(n, per_row, mid, d, c0, pitch):
    print("[case] copies, two slices", n, mid, d, flush=True)
    indptr, indices, values = _graph_with_hubs(n, per_row, seed=2)
    A, At, ws, wst = _build_in(_clean, indptr, indices, values, ISP_STAGE_MIN="1", ISP_MID_THRESHOLD=str(mid))
    assert (A.info()["spmm_pieces"] > 0) == (mid > 0)
    X, Xh = _operand(np.random.default_rng(d), n, d, d, 1)
    Y = torch.full((n, d), float("nan"), device="cuda")
    isp.spmm(A, X, Y)
    assert _holds_copy(ws, X, c0, pitch)
    assert_close(Y, *oracle.spmm(indptr, indices, values, Xh), "two slices of copies")
    ti, tj, _, tv = oracle.transpose(n, n, indptr, indices, values)
    isp.spmm(At, X, Y)
    assert _holds_copy(wst, X, c0, pitch)
    assert_close(Y, *oracle.spmm(ti, tj, tv, Xh), "two slices of copies, transpose")
    A.destroy()


def test_setting_is_the_sources():
    """ISP_STAGE_MIN is read when the matrix is built; its transpose and the room for its aliases follow, whatever is set by then."""
    n = 3000
    g = _graph_with_hubs(n, 20)
    for at_build, later in (("1", None), (None, "1"), ("1", "0")):
        print("[case] ISP_STAGE_MIN", at_build, later, flush=True)
        try:
            if at_build:
                os.environ["ISP_STAGE_MIN"] = at_build
            A = build(*g)
            os.environ.pop("ISP_STAGE_MIN", None)
            if later:
                os.environ["ISP_STAGE_MIN"] = later
            need = isp.csr_transpose_workspace(A)
            isp.csr_transpose_cached(A)
        finally:
            os.environ.pop("ISP_STAGE_MIN", None)
        assert isp.csr_transpose_workspace(A) == need
        rooms = isp.csr_alias_workspace(A, max_d=128) - isp.csr_alias_workspace(A, max_d=3)
        assert rooms == (2 * 4 * n * 128 if at_build else 0)  # (A's and the transpose's)
        A.destroy()


def test_more_workspace_than_asked_for_changes_nothing():
    """A transpose that shares its matrix's partitions takes copies by what the matrix asks for, not by what is left."""
    print("[case] larger workspace", flush=True)
    n, rng = 300_001, np.random.default_rng(0)
    i, j = rng.integers(0, n, 2_200_000), rng.integers(0, n, 2_200_000)
    code = np.unique(np.concatenate([i * n + j, j * n + i]))
    indptr = np.concatenate([[0], np.cumsum(np.bincount(code // n, minlength=n))]).astype(np.int64)
    g = indptr, (code % n).astype(np.int32), rng.standard_normal(code.size).astype(np.float32)
    rooms = []
    for more in (0, 512 * n + 4096):  # (the widest copies)
        A, At, _, _ = _build_in(lambda need: _clean(need + more), *g, ISP_STAGE_MIN="1", ISP_MID_THRESHOLD="0")
        assert A.info()["symmetric_pattern"] == 1
        rooms.append(isp.csr_alias_workspace(A, max_d=128) - isp.csr_alias_workspace(A, max_d=3))
        A.destroy()
    assert rooms[0] == rooms[1] == 0


def test_non_finite_rows_stay_where_they_are(graph):
    w, A, _, _ = graph
    print("[case] staged, one infinite row", flush=True)
    X = torch.ones(w.n, 50, device="cuda")
    j = int(w.indices[0])
    X[j] = float("inf")
    Y = torch.empty_like(X)
    isp.spmm(A, X, Y)
    rows = np.repeat(np.arange(w.n), np.diff(w.indptr))
    hit = np.zeros(w.n, dtype=bool)
    hit[rows[w.indices == j]] = True
    assert np.array_equal(~np.isfinite(Y.cpu().numpy()).all(1), hit)


def test_large_enough_by_itself():
    """The rule's own choice: 8 Mi entries, 32 and more per column, at a width whose rows cut a line more than they fill;
    forward and backward (a symmetric pattern of this size shares its partitions with the transpose)."""
    print("[case] staged by rule", flush=True)
    n, d, deg = 70_001, 20, 126
    rng = np.random.default_rng(0)
    half = rng.integers(1, n, (deg // 2,))
    off = np.unique(np.concatenate([half, n - half]))  # a circulant pattern: symmetric, distinct columns
    cols = np.sort((np.arange(n)[:, None] + off[None, :]) % n, axis=1).astype(np.int32)
    indptr = (np.arange(n + 1, dtype=np.int64) * off.size)
    vals = rng.standard_normal(n * off.size).astype(np.float32)
    assert indptr[-1] >= 8 << 20
    A = build(indptr, cols.reshape(-1), vals)
    At, _ = isp.csr_transpose_cached(A)
    assert A.info()["symmetric_pattern"] == 1
    Xh = rng.standard_normal((n, d)).astype(np.float32)
    X = torch.from_numpy(Xh).cuda()
    Y = torch.empty_like(X)
    isp.spmm(A, X, Y)
    assert_close(Y, *oracle.spmm(indptr, cols.reshape(-1), vals, Xh), "staged by rule")
    ti, tj, _, tv = oracle.transpose(n, n, indptr, cols.reshape(-1), vals)
    isp.spmm(At, X, Y)
    assert_close(Y, *oracle.spmm(ti, tj, tv, Xh), "staged by rule, transpose")
    A.destroy()


def test_same_bits_wherever_the_operand_lies():
    """Widths and pitches whose rows touch as many lines as their copies or more, by where the first row begins in one."""
    n, deg = 70_001, 126
    rng = np.random.default_rng(4)
    off = np.sort(rng.permutation(n)[:deg])
    cols = np.sort((np.arange(n)[:, None] + off[None, :]) % n, axis=1).astype(np.int32).reshape(-1)
    indptr = np.arange(n + 1, dtype=np.int64) * deg
    A = build(indptr, cols, rng.standard_normal(cols.size).astype(np.float32))
    for d, ld in ((40, 48), (132, 136), (140, 144), (192, 192), (270, 272)):
        print("[case] bases", d, ld, flush=True)
        X = torch.randn(n, d, device="cuda")
        first = None
        for shift in (0, 1, 5, 8, 14, 31):
            V = torch.empty(n * ld + shift + 32, device="cuda")[shift:shift + n * ld].view(n, ld)[:, :d]
            V.copy_(X)
            Y = isp.spmm(A, V, torch.empty(n, d, device="cuda"))
            first = Y if first is None else first
            assert torch.equal(first, Y), "base %d" % shift
    A.destroy()


def test_rule_on_a_packed_layout_that_the_transpose_shares():
    """The rule's own choice on a symmetric pattern with cut rows, 140 columns: 128 from one copy, 12 from the next."""
    print("[case] staged by rule, packed, shared", flush=True)
    n, d = 70_001, 140
    rng = np.random.default_rng(1)
    i, j = rng.integers(0, n, 4_700_000), rng.integers(0, n, 4_700_000)
    i[:9000] = np.repeat([3, 4, n - 1], 3000)
    code = np.unique(np.concatenate([i * n + j, j * n + i]))
    indptr = np.concatenate([[0], np.cumsum(np.bincount(code // n, minlength=n))]).astype(np.int64)
    indices, values = (code % n).astype(np.int32), rng.standard_normal(code.size).astype(np.float32)
    assert code.size >= 8 << 20
    vals = torch.from_numpy(values).cuda()
    ws = _clean(isp.csr_build_workspace(n, n, code.size))
    A = isp.csr_build(torch.from_numpy(indptr).cuda(), torch.from_numpy(indices).cuda(), vals, workspace=ws)
    At, _ = isp.csr_transpose_cached(A)
    assert A.info()["symmetric_pattern"] == 1 and A.info()["spmm_pieces"] == At.info()["spmm_pieces"] > 0
    Xh = rng.standard_normal((n, d)).astype(np.float32)
    X = torch.from_numpy(Xh).cuda()
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    for turn in range(2):
        isp.spmm(A, X, Y)
        assert _holds_copy(ws, X, 128, 16)
        isp.spmm_static_scratch(A, X, Z)
        assert torch.equal(Y, Z)
        assert_close(Y, *oracle.spmm(indptr, indices, values, Xh), "staged by rule, packed")
        ti, tj, _, tv = oracle.transpose(n, n, indptr, indices, values)
        isp.spmm(At, X, Y)
        isp.spmm_static_scratch(At, X, Z)
        assert torch.equal(Y, Z)
        assert_close(Y, *oracle.spmm(ti, tj, tv, Xh), "staged by rule, packed, transpose")
        values = rng.standard_normal(code.size).astype(np.float32)
        vals.copy_(torch.from_numpy(values))
        isp.csr_values_changed(A)
    A.destroy()
