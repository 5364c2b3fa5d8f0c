"""The work that users of this library give it, as measurable cases.

Graph operators on synthetic graphs of the sizes of the named workloads (workloads/graphs.py, workloads/hetero.py), made
on the GPU from a seed: SpMM on the hyb format (forward, and forward with the transposed product of a backward pass),
SpMM straight from CSR, the format conversion itself, SDDMM in CSR order and with a plan, and the relational
gather-matmul-scatter.  A graph has exactly `nnz` entries: degrees follow the named law, the columns of a row are
distinct, ascending and close to uniform.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2207_04606_amd as sptir

_SPMM_OPS = ("spmm", "spmm_train", "spmm_csr", "build")
_SDDMM_OPS = ("sddmm_csr", "sddmm_plan")


def _graph(name, op, rows, cols, nnz, feat, degrees, alpha, max_degree, values, parts, bucket):
    return {"name": name, "op": op, "rows": rows, "cols": cols, "nnz": nnz, "feat": feat, "degrees": degrees,
            "alpha": alpha, "max_degree": max_degree, "values": values, "parts": parts, "bucket": bucket}


def _relational(name, nodes, relations, nnz, d_in, d_out, workspace):
    return {"name": name, "op": "rgms", "nodes": nodes, "relations": relations, "nnz": nnz, "d_in": d_in,
            "d_out": d_out, "workspace": workspace}


def listed():
    return [
        # one layer of a citation network of a few thousand papers: launches and host work are all of it
        _graph("spmm_tiny", "spmm", 2708, 2708, 10556, 64, "power", 2.1, 2707, "inv_degree", 1, 5),
        # a training step's two products on a mid-sized citation network: Y = A X and dX = A^T dY
        _graph("spmm_train_medium", "spmm_train", 169343, 169343, 1166243, 128, "power", 2.0, 13000, "sym_norm", 4, 9),
        # a bipartite graph (sampled neighbours to targets) at the number of classes of the last layer: odd sizes, rows
        # of X that are not aligned to 16 bytes
        _graph("spmm_odd", "spmm", 50021, 61403, 1500007, 41, "power", 2.2, 5000, "uniform", 2, 6),
        # a protein association graph: long rows of like length, a value per edge
        _graph("spmm_protein", "spmm", 132534, 132534, 39561252, 128, "normal", 0.0, 7750, "uniform", 8, 10),
        # mean aggregation over a social network: the largest graph, a few very long rows
        _graph("spmm_social", "spmm", 232965, 232965, 114615892, 128, "power", 1.8, 21657, "inv_degree", 16, 11),
        # a graph that is used once (an inference batch): no decomposition pays, the product runs on CSR
        _graph("spmm_csr_medium", "spmm_csr", 169343, 169343, 1166243, 128, "power", 2.0, 13000, "sym_norm", 1, 9),
        # a graph that changes and is used once or twice: decomposed and multiplied
        _graph("build_medium", "build", 169343, 169343, 1166243, 64, "power", 2.0, 13000, "sym_norm", 4, 9),
        # edge scores of an attention layer, and the gradient of the edge values
        _graph("sddmm_csr_medium", "sddmm_csr", 169343, 169343, 1166243, 64, "power", 2.0, 13000, "uniform", 1, 9),
        # the same on the largest graph, whose structure is fixed: with a plan
        _graph("sddmm_plan_social", "sddmm_plan", 232965, 232965, 114615892, 128, "power", 1.8, 21657, "inv_degree", 0, 11),
        # relational graph convolutions: a small knowledge graph with wide features, a dense one, a large sparse one
        _relational("rgms_small", 27163, 46, 148100, 64, 64, False),
        _relational("rgms_dense", 93773, 51, 4762678, 32, 32, False),
        _relational("rgms_sparse", 1885136, 96, 5668682, 32, 32, False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("spmm", "spmm", "spmm", "spmm_train", "spmm_csr", "build", "sddmm_csr", "sddmm_plan", "rgms", "rgms"))
    if op == "rgms":
        nodes = _log_int(rng, 300, 1900000)
        relations = _log_int(rng, 5, 96)
        d_in, d_out = rng.choice(((32, 32), (32, 32), (64, 64), (64, 32), (128, 128), (128, 32)))
        nnz = min(int(nodes * math.exp(rng.uniform(math.log(3.0), math.log(50.0)))), 5600000 * 32 // d_in)
        nnz = max(nnz, relations)
        case = _relational("", nodes, relations, nnz, d_in, d_out, rng.random() < 0.25)
    else:
        rows = _log_int(rng, 2500, 235000)
        cols = rows if rng.random() < 0.6 else _log_int(rng, max(2500, rows // 3), min(235000, rows * 3))
        feat = _log_int(rng, 16, 256)
        kind = rng.random()
        feat = (feat + 31) // 32 * 32 if kind < 0.5 else (feat + 3) // 4 * 4 if kind < 0.75 else feat | 1
        mean = math.exp(rng.uniform(math.log(3.5), math.log(500.0)))
        most = 4.0e9 if op in ("spmm", "sddmm_plan") else 8.0e8
        if op in _SDDMM_OPS and feat % 4:
            most = 2.0e8
        nnz = int(min(rows * mean, rows * cols / 16.0, most / feat, 5.0e7))
        nnz = max(nnz, 3 * rows)
        # (degrees between 1 and a tenth of the columns, as in the listed graphs; short of that where rows are long)
        max_degree = min(cols - 1, max(cols // 10, 4 * (nnz // rows) + 8))
        degrees = rng.choice(("power", "power", "normal"))
        values = rng.choice(("inv_degree", "uniform", "sym_norm" if rows == cols else "uniform"))
        parts = min(16, 1 << max(0, (cols // 16384).bit_length()))
        if op == "sddmm_plan":
            parts = 0  # (chosen by the library)
        elif rng.random() < 0.3:
            parts = rng.choice((1, 2, 4, 8, 16))
        bucket = max(0, min(12, math.ceil(math.log2(nnz / rows)) + rng.choice((0, 0, 2, 3))))
        case = _graph("", op, rows, cols, nnz, feat, degrees, round(rng.uniform(1.8, 2.2), 2), max_degree, values, parts,
                      bucket)
    del case["name"]
    return case


# ----------------------------------------------------------------------------------------------------- inputs
def _fit_sum(deg, total, most):
    """Adds or takes 1 here and there until the degrees (1 .. most) sum to `total`."""
    while True:
        off = int(deg.sum()) - total
        if off == 0:
            return deg
        at = torch.nonzero(deg > 1 if off > 0 else deg < most).flatten()[:abs(off)]
        deg[at] += -1 if off > 0 else 1


def _degrees(case, gen):
    n, nnz, most = case["rows"], case["nnz"], case["max_degree"]
    if case["degrees"] == "normal":
        mean = nnz / n
        deg = torch.randn(n, generator=gen, device="cuda") * (mean / 3.0) + mean
        return _fit_sum(deg.round().clamp(1, most).long(), nnz, most)
    t = (1.0 - torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)) ** (-1.0 / (case["alpha"] - 1.0))
    lo, hi = 0.0, 2.0 * nnz / n
    for _ in range(40):
        mid = 0.5 * (lo + hi)
        if int((t * mid).floor_().clamp_(1, most).sum()) < nnz:
            lo = mid
        else:
            hi = mid
    return _fit_sum((t * hi).floor_().clamp_(1, most).long(), nnz, most)


def _csr(deg, n_cols, gen):
    """(indptr, indices, row of every entry): deg[r] distinct ascending columns per row."""
    n = deg.numel()
    indptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(deg, 0, out=indptr[1:])
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), deg)
    room = (n_cols + 1 - deg)[rows]  # a sorted draw from [0, n_cols - deg] plus 0, 1, 2, ... is strictly ascending
    key = (torch.rand(rows.numel(), generator=gen, device="cuda", dtype=torch.float64) * room).long().minimum(room - 1)
    key = torch.sort(rows * n_cols + key).values
    cols = key - rows * n_cols + (torch.arange(rows.numel(), device="cuda") - indptr[rows])
    return indptr.int(), cols.int(), rows


def _values(case, deg, rows, cols, gen):
    if case["values"] == "inv_degree":
        return (1.0 / deg.float())[rows]
    if case["values"] == "sym_norm":
        d = deg.double().rsqrt()
        return (d[rows] * d[cols.long()]).float()
    return 1.0 - torch.rand(rows.numel(), generator=gen, device="cuda")


def _prepare_relational(case, gen):
    n, n_rel, nnz = case["nodes"], case["relations"], case["nnz"]
    share = 1.0 / torch.arange(1, n_rel + 1, dtype=torch.float64, device="cuda") ** 0.8
    share = share[torch.randperm(n_rel, generator=gen, device="cuda")]
    per_rel = _fit_sum((share / share.sum() * nnz).floor_().clamp_(min=1).long(), nnz, nnz)
    popularity = 1.0 / (1.0 + torch.randperm(n, generator=gen, device="cuda").double()) ** 0.6
    cdf = torch.cumsum(popularity, 0)
    rel = torch.repeat_interleave(torch.arange(n_rel, device="cuda"), per_rel)
    at = torch.rand(nnz, generator=gen, device="cuda", dtype=torch.float64) * cdf[-1]
    stacked = rel * n + torch.searchsorted(cdf, at).clamp_(max=n - 1)
    count = torch.bincount(stacked, minlength=n_rel * n).clamp_(max=n)
    short = nnz - int(count.sum())  # (only where a node is drawn more often than there are nodes)
    if short > 0:
        count[torch.nonzero(count == 0).flatten()[:short]] += 1
    indptr, indices, rows = _csr(count, n, gen)
    values = (1.0 / count.float())[rows]
    state = {"op": "rgms",
             "handle": sptir.sptir_rgms_build(n_rel, n, n, indptr, indices, values, -1,
                                              case["d_out"] if case["workspace"] else 0),
             "X": torch.randn(n, case["d_in"], generator=gen, device="cuda"),
             "W": torch.randn(n_rel, case["d_in"], case["d_out"], generator=gen, device="cuda") / math.sqrt(case["d_in"]),
             "Y": torch.empty(n, case["d_out"], device="cuda")}
    return state


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["op"] == "rgms":
        return _prepare_relational(case, gen)
    op, m, n, feat = case["op"], case["rows"], case["cols"], case["feat"]
    deg = _degrees(case, gen)
    indptr, indices, rows = _csr(deg, n, gen)
    values = _values(case, deg, rows, indices, gen)
    state = {"op": op, "shape": (m, n), "hyb": (case["parts"], case["bucket"])}
    if op != "spmm":
        state["csr"] = (indptr, indices, values)
    if op in _SDDMM_OPS:
        state["X"] = torch.randn(m, feat, generator=gen, device="cuda")
        state["Yt"] = torch.randn(n, feat, generator=gen, device="cuda")
        state["B"] = torch.empty_like(values)
        if op == "sddmm_plan":
            state["plan"] = sptir.sptir_sddmm_plan_build(m, n, indptr, indices, case["parts"], feat)
        return state
    state["X"] = torch.randn(n, feat, generator=gen, device="cuda")
    state["Y"] = torch.empty(m, feat, device="cuda")
    if op in ("spmm", "spmm_train"):
        state["A"] = sptir.sptir_hyb_build(m, n, indptr, indices, values, case["parts"], case["bucket"])
    if op == "spmm_train":
        order = torch.argsort(indices.long() * m + rows)
        indptr_t = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(torch.bincount(indices, minlength=n), 0, out=indptr_t[1:])
        state["At"] = sptir.sptir_hyb_build(n, m, indptr_t.int(), rows[order].int(), values[order], case["parts"],
                                            case["bucket"])
        state["dY"] = torch.randn(m, feat, generator=gen, device="cuda")
        state["dX"] = torch.empty(n, feat, device="cuda")
    return state


# -------------------------------------------------------------------------------------------------- one pass
def run(state):
    op = state["op"]
    if op == "rgms":
        sptir.sptir_rgms(state["handle"], state["X"], state["W"], state["Y"])
        return state["Y"]
    if op == "spmm":
        sptir.sptir_spmm(state["A"], state["X"], state["Y"])
        return state["Y"]
    if op == "spmm_train":
        sptir.sptir_spmm(state["A"], state["X"], state["Y"])
        sptir.sptir_spmm(state["At"], state["dY"], state["dX"])
        return [state["Y"], state["dX"]]
    if op == "sddmm_plan":
        sptir.sptir_sddmm(state["plan"], state["csr"][2], state["X"], state["Yt"], state["B"])
        return state["B"]
    m, n = state["shape"]
    if op == "sddmm_csr":
        sptir.sptir_sddmm_csr(m, n, *state["csr"], state["X"], state["Yt"], state["B"])
        return state["B"]
    if op == "spmm_csr":
        sptir.sptir_spmm_csr(m, n, *state["csr"], state["X"], state["Y"])
        return state["Y"]
    hyb = sptir.sptir_hyb_build(m, n, *state["csr"], *state["hyb"])
    sptir.sptir_spmm(hyb, state["X"], state["Y"])
    hyb.destroy()
    return state["Y"]


def _expected_pairs(case):
    """Expected number of (relation, row) pairs with an entry: what the product with W cannot do without."""
    n, n_rel = case["nodes"], case["relations"]
    share = 1.0 / np.arange(1, n_rel + 1) ** 0.8
    edges = share / share.sum() * case["nnz"]
    at = np.unique(np.geomspace(1, n, 2000).round())  # ranks, each standing for those up to the next
    many = np.diff(np.append(at, n + 1))
    weight = 1.0 / at ** 0.6
    p = weight / (weight * many).sum()
    return float((many * (1.0 - np.exp(-edges[:, None] * p))).sum())


def work(case):
    nnz = case["nnz"]
    if case["op"] == "rgms":
        n, n_rel, d_in, d_out = case["nodes"], case["relations"], case["d_in"], case["d_out"]
        return {"bytes": 8 * nnz + 4 * n * (d_in + d_out) + 4 * n_rel * d_in * d_out,
                "flops": 2 * nnz * d_in + 2 * _expected_pairs(case) * d_in * d_out}
    m, n, feat = case["rows"], case["cols"], case["feat"]
    dense = 4 * feat * (m + n)
    if case["op"] in _SDDMM_OPS:
        return {"bytes": 12 * nnz + 4 * (m + 1) + dense, "flops": 2 * nnz * feat}
    passes = 2 if case["op"] == "spmm_train" else 1
    return {"bytes": passes * (8 * nnz + 4 * (m + 1) + dense), "flops": passes * 2 * nnz * feat}


def tolerance(case):
    # float32 sums and products in another order
    return {"rel": 1e-5, "max": 1e-3}
