"""The work that users of the sparse GNN operations have them do, as measurable cases.

A case is one training or inference step's sparse part on one seeded synthetic graph.  `op` says which:

  infer      Y = A X                                           (inference of one aggregation)
  train      Y = A X and dX = A^T dY                           (a GCN / GIN layer's forward and backward)
  layer      the same through the torch.autograd wrapper       (as it sits inside a PyTorch model)
  edges      trained edge weights: new values, Y = A X, dX = A^T dY, dA = SDDMM(dY, X)
  sddmm      one dot product per stored entry                  (edge scoring)
  mean, max  matmul(A, X, reduce) and its backward             (GraphSAGE aggregators)
  fused      FusedMM with the sigmoid, forward and backward    (graph embedding)
  new_graph  a graph seen once: handle, transpose, forward and backward   (sampled mini-batches)

Everything but `new_graph` keeps the handle with its cached transpose, as a program that trains for many epochs does.
Graphs are R-MAT (quadrants .57 / .19 / .19 / .05, vertices relabelled at random) or uniform, without duplicate
entries, rows column-sorted, with exactly `nnz` stored entries; all arrays are fp32 / int32 / int64 as the library takes them.
"""
import math

import torch

import paper_2403_14853_amd as isp
from paper_2403_14853_amd import autograd as isp_autograd

# Passes over the entries that each op makes (what a case costs, next to nnz and d).
PASSES = {"infer": 1, "train": 2, "layer": 2, "edges": 3, "sddmm": 1, "mean": 2, "max": 2, "fused": 4, "new_graph": 2}
BACKWARD = ("train", "layer", "edges", "mean", "max", "fused")  # ops that use the cached transpose
MAX_NNZ, MAX_COST = 120_000_000, 30e9


def _case(name, op, graph, n, nnz, d, values="unit", symmetric=True, n_cols=0):
    return {"name": name, "op": op, "graph": graph, "n": n, "n_cols": n_cols or n, "nnz": nnz, "d": d, "values": values,
            "symmetric": symmetric}


def listed():
    return [
        # one aggregation on a small molecule- or citation-sized graph: latency and launches are all there is
        _case("small-infer-d32", "infer", "er", 4_096, 36_864, 32, "gcn", symmetric=False),
        # a layer of a small node-classification model, hidden width 16, inside PyTorch
        _case("citation-layer-d16", "layer", "rmat", 19_717, 108_365, 16, "gcn"),
        # a hidden GCN layer on a mid-sized citation graph (the repository's benchmark configuration 1)
        _case("arxiv-layer-d128", "layer", "rmat", 169_343, 2_404_585, 128, "gcn"),
        # the output layer of the same model: as many columns as there are classes, which is rarely a round number
        _case("arxiv-train-d47", "train", "rmat", 169_343, 2_404_585, 47, "gcn"),
        # first-layer aggregation of raw node features (602 wide, no gradient needed) on a dense social graph
        _case("dense-infer-d602", "infer", "rmat", 232_965, 114_600_001, 602, "rowmean"),
        # trained edge weights on the same graph (configuration 2 with the values rewritten in every step)
        _case("dense-edges-d128", "edges", "rmat", 232_965, 114_600_001, 128, "rowmean"),
        # the largest power-law graph, a hidden layer (configuration 3)
        _case("products-train-d128", "train", "rmat", 2_449_029, 123_629_211, 128, "gcn"),
        # max aggregation of 100-wide features on a graph of a third of that size
        _case("products-max-d100", "max", "rmat", 800_003, 40_000_003, 100),
        # embedding of a directed graph, half of the rows empty (configuration 4)
        _case("embed-fused-d64", "fused", "rmat", 1_048_576, 16_851_165, 64, symmetric=False),
        # the same operation at a width that is no multiple of 4
        _case("embed-fused-d50", "fused", "rmat", 300_007, 3_000_001, 50),
        # mini-batch training: every batch is a new, mid-sized sampled graph, mean aggregation as edge values
        _case("minibatch-new-graph-d64", "new_graph", "rmat", 100_003, 1_000_001, 64, "rowmean", symmetric=False),
        # scoring the entries of a rectangular (user x item) matrix
        _case("bipartite-sddmm-d64", "sddmm", "rmat", 500_009, 8_000_003, 64, symmetric=False, n_cols=120_011),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choice(sorted(PASSES))
    graph = "rmat" if rng.random() < 0.8 else "er"
    n = int(_log_uniform(rng, 1_000, 2_500_000))
    n_cols = n
    if op in ("infer", "sddmm") and rng.random() < 0.3:
        n_cols = int(_log_uniform(rng, max(1_000, n / 8), min(2_500_000, n * 8)))
    d = int(_log_uniform(rng, 8, 256 if op == "fused" else 602))
    if rng.random() < 0.5:  # hidden widths are usually round, feature and class counts are not
        d = (d + 7) // 8 * 8
    symmetric = n_cols == n and rng.random() < 0.6
    # average row lengths from 4 to 500; denser than the square root of the size only the small world is
    nnz = n * _log_uniform(rng, 4, min(500, math.sqrt(min(n, n_cols))))
    nnz = int(min(nnz, MAX_NNZ, MAX_COST / (PASSES[op] * (d + 16)), 16e6 if op == "new_graph" else nnz))
    if nnz < 3 * n:  # the largest sizes: fewer vertices rather than no edges
        n_cols = max(1_000, int(n_cols * nnz / (3 * n)))
        n = max(1_000, nnz // 3)
        n_cols = n if symmetric or op not in ("infer", "sddmm") else n_cols
    values = rng.choice(["unit", "gcn", "rowmean"]) if n_cols == n else "unit"
    if op == "edges" and values == "unit":
        values = "rowmean"
    case = _case("", op, graph, n, nnz, d, values, symmetric, n_cols)
    del case["name"]
    return case


# ---- graphs -------------------------------------------------------------------------------------------------
def _rmat_pairs(m, levels, n, n_cols, g):
    """m candidate (row, column) pairs; a pair that falls outside the matrix is given up for another draw's sake."""
    out = []
    while m > 0:
        k = min(m, 1 << 24)
        u = torch.zeros(k, dtype=torch.int32, device="cuda")
        v = torch.zeros(k, dtype=torch.int32, device="cuda")
        for _ in range(levels):
            r = torch.rand(k, device="cuda", generator=g)
            u.mul_(2).add_(r >= 0.76)
            v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
        if n_cols != n:
            u, v = u % n, v % n_cols
        keep = (u < n) & (v < n_cols)
        out.append((u[keep], v[keep]))
        m -= k
    return torch.cat([a for a, _ in out]), torch.cat([b for _, b in out])


def _graph(case, seed):
    """(indptr, indices): exactly nnz distinct entries, rows column-sorted.  A symmetric graph has every vertex's own loop
    and pairs (u, v), (v, u); it falls short of an odd remainder by leaving out one vertex's loop."""
    n, n_cols, nnz = case["n"], case["n_cols"], case["nnz"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    sym = case["symmetric"]
    loops = 0
    want = nnz
    if sym:
        loops = n - ((nnz - n) & 1)
        want = (nnz - loops) // 2
    levels = max(1, math.ceil(math.log2(max(n, n_cols))))
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    for turn in range(12):
        missing = want - keys.numel()
        if missing <= 0:
            break
        m = int(missing * 1.25) + 1024
        if case["graph"] == "rmat" and turn < 8:
            u, v = _rmat_pairs(m * 2, levels, n, n_cols, g)
        else:
            u = torch.randint(n, (m,), device="cuda", generator=g, dtype=torch.int32)
            v = torch.randint(n_cols, (m,), device="cuda", generator=g, dtype=torch.int32)
        if n_cols == n:
            keep = u != v
            u, v = u[keep], v[keep]
        if sym:
            u, v = torch.minimum(u, v), torch.maximum(u, v)
        keys = torch.unique(torch.cat([keys, u.long() * n_cols + v]))
    extra = keys.numel() - want
    if extra > 0:  # leave a random choice of the entries out
        keep = torch.ones(keys.numel(), dtype=torch.bool, device="cuda")
        keep[torch.randperm(keys.numel(), device="cuda", generator=g)[:extra]] = False
        keys = keys[keep]
    u, v = keys // n_cols, keys % n_cols
    if case["graph"] == "rmat":  # popular vertices do not sit next to each other
        pu = torch.randperm(n, device="cuda", generator=g)
        pv = pu if n_cols == n else torch.randperm(n_cols, device="cuda", generator=g)
        u, v = pu[u], pv[v]
    keys = u * n_cols + v
    if sym:
        own = torch.arange(loops, device="cuda")
        keys = torch.cat([keys, v * n_cols + u, own * n_cols + own])
    keys = torch.sort(keys).values
    u = keys // n_cols
    indices = (keys - u * n_cols).to(torch.int32)
    indptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    indptr[1:] = torch.cumsum(torch.bincount(u, minlength=n), 0)
    return indptr, indices


def _values(case, indptr, indices, g):
    if case["values"] == "unit":
        return None
    deg = (indptr[1:] - indptr[:-1]).clamp(min=1).float()
    rows = torch.repeat_interleave(torch.arange(case["n"], device="cuda", dtype=torch.int32), indptr[1:] - indptr[:-1])
    if case["values"] == "gcn":
        s = deg.rsqrt()
        return s[rows] * s[indices]
    return (1.0 / deg)[rows]


# ---- what perf measures ---------------------------------------------------------------------------------------
def prepare(case, seed):
    op, n, n_cols, d = case["op"], case["n"], case["n_cols"], case["d"]
    indptr, indices = _graph(case, seed)
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    values = _values(case, indptr, indices, g)

    def features(rows, std=1.0):
        return torch.randn(rows, d, device="cuda", generator=g) * std

    s = {"op": op, "indptr": indptr, "indices": indices, "values": values, "n_cols": n_cols,
         "X": features(n_cols, 0.1 if op == "fused" else 1.0)}
    if op != "infer":
        s["dY"] = features(n)
    if op in ("layer", "mean", "max"):
        s["graph"] = isp_autograd.SparseGraph(indptr, indices, values, n_cols=n_cols)
        s["graph"].transpose()
        s["X"].requires_grad_(True)
    elif op != "new_graph":
        s["A"] = isp.csr_build(indptr, indices, values, n_cols=n_cols)
        if op in BACKWARD:
            s["At"] = isp.csr_transpose_cached(s["A"])[0]
    if op in ("infer", "train", "edges", "fused"):
        s["Y"] = torch.empty(n, d, device="cuda")
    if op in ("train", "edges", "fused"):
        s["dX"] = torch.empty(n_cols, d, device="cuda")
    if op in ("edges", "sddmm"):
        s["dA"] = torch.empty(case["nnz"], device="cuda")
    if op == "edges":  # the weights that the rest of the model hands over in every step
        s["weights"] = values * (0.5 + torch.rand(case["nnz"], device="cuda", generator=g))
    return s


def run(s):
    op, X = s["op"], s["X"]
    if op == "infer":
        return isp.spmm(s["A"], X, s["Y"])
    if op == "train":
        return isp.spmm(s["A"], X, s["Y"]), isp.spmm(isp.csr_transpose_cached(s["A"])[0], s["dY"], s["dX"])
    if op in ("layer", "mean", "max"):
        Y = isp_autograd.matmul(s["graph"], X, "sum" if op == "layer" else op)
        return Y, torch.autograd.grad(Y, X, s["dY"])[0]
    if op == "edges":
        s["values"].copy_(s["weights"])
        isp.csr_values_changed(s["A"])
        isp.spmm(s["A"], X, s["Y"])
        isp.spmm(isp.csr_transpose_cached(s["A"])[0], s["dY"], s["dX"])
        return s["Y"], s["dX"], isp.sddmm(s["A"], s["dY"], X, s["dA"])
    if op == "sddmm":
        return isp.sddmm(s["A"], s["dY"], X, s["dA"])
    if op == "fused":
        return isp.fusedmm(s["A"], X, s["Y"]), isp.fusedmm_backward(s["A"], X, s["dY"], s["dX"])
    A = isp.csr_build(s["indptr"], s["indices"], s["values"], n_cols=s["n_cols"])
    Y = isp.spmm(A, X, torch.empty_like(s["dY"]))
    return Y, isp.spmm(isp.csr_transpose_cached(A)[0], s["dY"], torch.empty_like(X))


def work(case):
    op, n, n_cols, nnz, d = case["op"], case["n"], case["n_cols"], case["nnz"], case["d"]
    entry = 4 if case["values"] == "unit" else 8
    csr = 8 * (n + 1) + entry * nnz
    csr_t = 8 * (n_cols + 1) + entry * nnz
    out, inp = 4 * n * d, 4 * n_cols * d  # Y-shaped and X-shaped matrices
    mul = 2.0 * nnz * d
    if op == "infer":
        return {"bytes": csr + inp + out, "flops": mul}
    if op in ("train", "layer", "mean"):
        return {"bytes": csr + csr_t + 2 * inp + 2 * out, "flops": 2 * mul}
    if op == "max":  # the winning positions are written by the forward and read by the backward
        return {"bytes": csr + csr_t + 2 * inp + 2 * out + 2 * out, "flops": 2 * mul}
    if op == "edges":  # weights copied in, permuted into the transpose's order, gradients out
        return {"bytes": 3 * csr + 2 * inp + 2 * out + inp + out + 4 * nnz * 5, "flops": 3 * mul}
    if op == "sddmm":
        return {"bytes": 8 * (n + 1) + 4 * nnz + inp + out + 4 * nnz, "flops": mul}
    if op == "fused":  # scores once forward, again with two further products per entry backward
        return {"bytes": csr + inp + out + csr + csr_t + 2 * inp + out, "flops": 7 * mul}
    return {"bytes": 2 * csr + 2 * csr_t + 4 * nnz + 2 * inp + 2 * out, "flops": 2 * mul}


def tolerance(case):
    return {"rel": 1e-5}  # fp32 sums of fp32 products in another order; positions and signs of max are exact
