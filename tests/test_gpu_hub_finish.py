"""Hub rows that the launch of their segments puts together: numbers of segments around the quarters in which they are added, every
lane shape, both column slices, more segments than the rule takes; several calls in a row (the counters start over by themselves),
bit-identical through an alias, whose hub rows a fix-up launch adds, and within tolerance of the oracle."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2403_14853_amd as isp
from gpu_util import assert_close, build, dev

pytestmark = pytest.mark.gpu

ENV = {"ISP_HUB_THRESHOLD": "16", "ISP_SEGMENT_LEN": "8", "ISP_BANDS": "1", "ISP_MID_THRESHOLD": "0"}


def _graph(hub_lengths, n_rows, n_cols, seed, square=False):
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 5, n_rows)
    deg[rng.permutation(n_rows)[:len(hub_lengths)]] = hub_lengths
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    rows = np.repeat(np.arange(n_rows), deg)
    cols = rng.integers(0, n_cols, len(rows))
    if square:  # most entries of the transpose in hub rows too
        hot = rng.integers(0, 40, len(rows))
        cols = np.where(rng.random(len(rows)) < 0.7, hot * (n_cols // 40), cols)
    cols = cols[np.lexsort((cols, rows))].astype(np.int32)
    values = rng.standard_normal(len(rows)).astype(np.float32)
    saved = {k: os.environ.get(k) for k in ENV}
    os.environ.update(ENV)
    try:
        A = build(indptr, cols, values, n_cols=n_cols)
        isp.csr_transpose_cached(A)
    finally:
        for k, v in saved.items():
            if v is None:
                os.environ.pop(k)
            else:
                os.environ[k] = v
    return indptr, cols, values, A, isp.csr_alias(A, max_d=320)


FEW = list(range(17, 330, 8)) + [17, 20, 24, 25, 2_000, 2_001, 4_099]  # 3 to 513 segments: the longest row is too long
MANY = [24] * 3_000
# The longest row as long as the launches with 64, 32 and up to 16 lanes to a group finish, and a segment longer.
SHORT = list(range(17, 330, 8)) + [17, 20, 24, 25, 504, 512, 761, 768]  # 3 to 96 segments: every launch
WIDE, WIDER = SHORT + [1_024], SHORT + [1_025]                # 128 and 129
LONG, LONGER = SHORT + [1_024, 4_096], SHORT + [1_024, 4_097]  # 512 and 513


@pytest.mark.parametrize("hubs, n_cols, widths", [
    (FEW, 700, [3, 4, 16, 17, 32, 64, 65, 100, 128, 130, 200, 256, 301]),
    (FEW, 82_000, [127, 128, 256]),   # 128 whole-line columns run as two slices
    (SHORT, 700, [3, 4, 16, 17, 32, 64, 65, 100, 128, 130, 200, 256, 301]),
    (SHORT, 82_000, [127, 128, 200, 256]),
    (WIDE, 700, [64, 65, 128, 130, 256]),
    (WIDER, 700, [64, 65, 128, 130]),
    (LONG, 700, [8, 30, 64, 100]),
    (LONGER, 700, [8, 30, 64, 100]),
    (MANY, 700, [8, 64, 100, 256]),
])
def test_spmm_and_mean(hubs, n_cols, widths):
    indptr, cols, values, A, B = _graph(hubs, 4_000, n_cols, len(hubs) + n_cols)
    info = A.info()
    assert info["n_segments"] == sum((h + 7) // 8 for h in hubs) and (info["n_segments"] > 8_192) == (hubs is MANY)
    length = np.maximum(np.diff(indptr), 1)[:, None]
    for d in widths:
        print("[case] %d segments, %d columns, d = %d" % (info["n_segments"], n_cols, d), flush=True)
        for turn in range(3):
            X = np.random.default_rng(10 * d + turn).standard_normal((n_cols, d)).astype(np.float32)
            Xd = dev(X)
            Y, Z = (torch.full((4_000, d), float("nan"), device="cuda") for _ in range(2))
            isp.spmm(A, Xd, Y)
            isp.spmm(B, Xd, Z)
            assert torch.equal(Y, Z)
            ref, mag = oracle.spmm(indptr, cols, values, X)
            assert_close(Y, ref, mag, "spmm")
            isp.spmm_reduce(A, Xd, Y, "mean")
            isp.spmm_reduce(B, Xd, Z, "mean")
            assert torch.equal(Y, Z)
            assert_close(Y, ref / length, mag / length, "mean")
    A.destroy()


@pytest.mark.parametrize("hubs", [FEW, MANY, SHORT, WIDE, LONG])
def test_fusedmm(hubs):
    n = 4_000
    indptr, cols, values, A, B = _graph(hubs, n, n, 5, square=True)
    for d in (4, 16, 30, 64, 65, 128, 200, 256):
        print("[case] fusedmm, %d hub rows, d = %d" % (len(hubs), d), flush=True)
        for turn in range(2):
            rng = np.random.default_rng(10 * d + turn)
            X = (0.2 * rng.standard_normal((n, d))).astype(np.float32)
            G = rng.standard_normal((n, d)).astype(np.float32)
            Xd, Gd = dev(X), dev(G)
            Y, Z = (torch.full((n, d), float("nan"), device="cuda") for _ in range(2))
            isp.fusedmm(A, Xd, Y)
            isp.fusedmm(B, Xd, Z)
            assert torch.equal(Y, Z)
            assert_close(Y, *oracle.fusedmm(indptr, cols, values, X), "fusedmm")
            isp.fusedmm_backward(A, Xd, Gd, Y)
            isp.fusedmm_backward(B, Xd, Gd, Z)
            assert torch.equal(Y, Z)
            assert_close(Y, *oracle.fusedmm_backward(indptr, cols, values, X, G), "fusedmm backward")
    A.destroy()


@pytest.mark.parametrize("hubs", [FEW, MANY])
def test_min_and_max(hubs):
    """Forward bit for bit (ties to the first entry), backward bit-identical through an alias and within tolerance."""
    n = 4_000
    indptr, cols, values, A, B = _graph(hubs, n, n, 9, square=True)
    for d in (4, 30, 32, 64, 65, 100, 128, 131, 256):
        for reduce in ("min", "max"):
            print("[case] %s, %d hub rows, d = %d" % (reduce, len(hubs), d), flush=True)
            for turn in range(2):
                rng = np.random.default_rng(10 * d + turn)
                X = rng.integers(-8, 9, (n, d)).astype(np.float32)  # (many ties)
                G = rng.standard_normal((n, d)).astype(np.float32)
                Xd, Gd = dev(X), dev(G)
                Y, Z, dX, dZ = (torch.full((n, d), float("nan"), device="cuda") for _ in range(4))
                arg, arg_b = (torch.full((n, d), -7, dtype=torch.int32, device="cuda") for _ in range(2))
                isp.spmm_reduce(A, Xd, Y, reduce, arg)
                isp.spmm_reduce(B, Xd, Z, reduce, arg_b)
                ref, ref_arg, _ = oracle.spmm_reduce(indptr, cols, values, X, reduce)
                assert torch.equal(Y, Z) and torch.equal(arg, arg_b)
                assert np.array_equal(Y.cpu().numpy(), ref) and np.array_equal(arg.cpu().numpy(), ref_arg)
                isp.spmm_reduce_backward(A, Gd, dX, reduce, arg)
                isp.spmm_reduce_backward(B, Gd, dZ, reduce, arg)
                assert torch.equal(dX, dZ)
                want, mag = oracle.spmm_reduce_backward(n, indptr, cols, values, G, reduce, ref_arg)
                assert_close(dX, want, mag, "backward")
    A.destroy()


def _pairs(lengths, n, seed):
    """Hub rows of these lengths, rows of 100 to 160 entries, which let the launch finish its hub rows, and rows of 0 to 5."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 6, n)
    rows = rng.permutation(n)
    deg[rows[:len(lengths)]] = lengths
    deg[rows[len(lengths):len(lengths) + 60]] = rng.integers(100, 161, 60)
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    owner = np.repeat(np.arange(n), deg)
    cols = rng.integers(0, n, len(owner))
    cols = cols[np.lexsort((cols, owner))].astype(np.int32)
    values = rng.integers(1, 4, len(owner)).astype(np.float32)
    env = {"ISP_HUB_THRESHOLD": "160", "ISP_SEGMENT_LEN": "80", "ISP_BANDS": "1"}
    saved = {k: os.environ.get(k) for k in env}
    os.environ.update(env)
    try:
        dv = dev(values)
        A = isp.csr_build(dev(indptr), dev(cols), dv, n_cols=n)
    finally:
        for k, v in saved.items():
            if v is None:
                os.environ.pop(k)
            else:
                os.environ[k] = v
    return indptr, cols, values, dv, A, np.sort(rows[:len(lengths)])


@pytest.mark.parametrize("d, n", [(4, 6_000), (16, 6_000), (30, 6_000), (32, 6_000), (33, 6_000), (64, 6_000), (65, 6_000), (100, 6_000), (128, 6_000), (131, 6_000),
                                  (4, 190_000), (11, 190_000), (16, 190_000)])
def test_min_and_max_in_the_launch_of_the_segments(d, n):
    """The forward that finishes its hub rows, up to as many segments as it folds: bit for bit with the oracle (ties to the first entry),
    and with the fix-up launch (an alias) also where products are NaN: a row's first entry, a later segment's first, a whole
    segment, all segments of a lane group's part, everything but the row's end."""
    many = n > 6_000  # (entries enough for four lanes to a row)
    lanes = 4 if many else 8 if d <= 32 else 16 if d <= 64 else 32
    limit = 96 if lanes <= 8 else 32  # segments of the longest row
    lengths = [80 * s - k for s in range(3, limit + 1, limit // 10) for k in (0, 79)] + [80 * limit] * 3
    lengths = [h for h in lengths if h > 160]
    indptr, cols, values, dv, A, hubs = _pairs(lengths, n, d)
    info = A.info()
    assert (info["nnz"] >= 512 << 10) == many
    slots = 16 * torch.cuda.get_device_properties(0).multi_processor_count
    assert info["n_segments"] == sum((h + 79) // 80 for h in lengths) and 3 * info["n_segments"] <= slots
    assert 2 * info["bin_nnz"][3] >= info["segment_len"] * info["bin_rows"][3] > 0
    rng = np.random.default_rng(d)
    X = rng.integers(-8, 9, (n, d)).astype(np.float32)  # (many ties)
    nan = values.copy()
    for i, r in enumerate(hubs):
        a, b = indptr[r], indptr[r + 1]
        n_seg = -(-(b - a) // 80)
        part = -(-n_seg // (64 // lanes))
        first, last = [(0, 1), (80, 81), (0, 80), (80, 160), (80 * part, 160 * part), (0, b - a - 1)][i % 6]
        nan[a + first:min(a + last, b)] = np.nan
    Xd = dev(X)
    for with_nan in (False, True):
        if with_nan:
            dv.copy_(dev(nan))
            isp.csr_values_changed(A)
        B = isp.csr_alias(A, max_d=d)
        for reduce in ("min", "max"):
            print("[case] %s, d = %d, %d segments, nan: %d" % (reduce, d, info["n_segments"], with_nan), flush=True)
            for turn in range(2):  # (the counters start over by themselves)
                Y, Z = (torch.full((n, d), 7.5, device="cuda") for _ in range(2))
                arg, arg_b = (torch.full((n, d), -7, dtype=torch.int32, device="cuda") for _ in range(2))
                isp.spmm_reduce(A, Xd, Y, reduce, arg)
                isp.spmm_reduce(B, Xd, Z, reduce, arg_b)
                assert torch.equal(Y.view(torch.int32), Z.view(torch.int32)) and torch.equal(arg, arg_b)
            if with_nan:
                assert torch.isnan(Y[torch.from_numpy(hubs).cuda()]).any()
            else:
                ref, ref_arg, _ = oracle.spmm_reduce(indptr, cols, values, X, reduce)
                assert np.array_equal(Y.cpu().numpy(), ref) and np.array_equal(arg.cpu().numpy(), ref_arg)
        B.destroy()
    A.destroy()
