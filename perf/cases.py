"""Performance cases: the calls a program makes into this library, over the
sizes it is used at.

Every case names a call and a sparsity pattern.

Calls:
* ``spmm``     one ``sd_spmm`` on a plan the program keeps (the plan is made
               once per matrix and reused, so it belongs to ``prepare``);
* ``noalloc``  one ``sd_spmm_merge_noalloc`` straight from a device CSR, for
               programs that may not allocate (graph capture, serving loops);
* ``refresh``  a new matrix every pass: ``sd_plan_device`` on a CSR in device
               memory, one ``sd_spmm``, the plan destroyed (sampled or rebuilt
               graphs, re-assembled operators);
* ``epoch``    one full-batch training step of the two-layer GCN.

Patterns: ``uniform`` rows, ``stencil`` (7-point Laplacian), ``ragged`` rows
around a band, R-MAT ``graph`` with GCN values, ``blocks`` of 16x16.  All are
drawn on the GPU from the seed with torch.
"""
from __future__ import annotations

import math

import torch

import paper_2608_05033_amd as sd
from paper_2608_05033_amd import gcn

DEV = "cuda:0"


# ------------------------------------------------------------------ cases ---
def listed():
    return [
        # a small operator applied to a narrow block of vectors: launch latency
        {"name": "uniform_1k_n32", "call": "spmm", "pattern": "uniform", "m": 1024, "k": 1024, "row": 8, "n": 32,
         "transpose": False},
        # a stencil operator on a cube, times a block of 64 vectors
        {"name": "stencil_64_n64", "call": "spmm", "pattern": "stencil", "nx": 64, "ny": 64, "nz": 64, "n": 64,
         "transpose": False},
        # the matrix-vector product of an iterative solver, on an odd grid
        {"name": "stencil_odd_n1", "call": "spmm", "pattern": "stencil", "nx": 127, "ny": 61, "nz": 83, "n": 1,
         "transpose": False},
        # an unstructured mesh: ragged rows near a band, no row long enough to split
        {"name": "ragged_n96", "call": "spmm", "pattern": "ragged", "m": 300007, "k": 300007, "mean": 24.0,
         "sigma": 0.6, "band": 20000, "n": 96, "transpose": False},
        # a web or social graph times wide features
        {"name": "graph_1m_n128", "call": "spmm", "pattern": "graph", "scale": 20, "verts": 1 << 20,
         "edges": 16 << 20, "n": 128, "transpose": False},
        # the same graph, a narrow block (label propagation, a few personalised vectors)
        {"name": "graph_1m_n8", "call": "spmm", "pattern": "graph", "scale": 20, "verts": 1 << 20,
         "edges": 16 << 20, "n": 8, "transpose": False},
        # the backward aggregation of a full-batch GCN on the largest graph
        {"name": "graph_2m4_bwd_n64", "call": "spmm", "pattern": "graph", "scale": 22, "verts": 2400000,
         "edges": 62000000, "n": 64, "transpose": True},
        # a whole training step of the two-layer GCN on a middling graph
        {"name": "gcn_epoch_262k", "call": "epoch", "pattern": "graph", "scale": 18, "verts": 1 << 18,
         "edges": 4 << 20, "feats": 128, "hidden": 128, "classes": 64},
        # a block-sparse operator (16x16 tiles nearly full) times 64 vectors
        {"name": "blocks_8192_n64", "call": "spmm", "pattern": "blocks", "m": 131072, "k": 131072, "row": 32,
         "window": 512, "fill": 0.9, "n": 64, "transpose": False},
        # a smaller block operator with ragged edges and a width of no whole tile
        {"name": "blocks_odd_n100", "call": "spmm", "pattern": "blocks", "m": 24011, "k": 23003, "row": 21,
         "window": 200, "fill": 0.88, "n": 100, "transpose": False},
        # a graph product from a serving loop that may not allocate
        {"name": "noalloc_graph_n32", "call": "noalloc", "pattern": "graph", "scale": 18, "verts": 200003,
         "edges": 3000000, "n": 32},
        # a graph that changes every step: plan on the device, one product
        {"name": "refresh_graph_n64", "call": "refresh", "pattern": "graph", "scale": 19, "verts": 500009,
         "edges": 8000000, "n": 64, "transpose": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, most):
    """Dense widths in use: powers of two, multiples of 4, odd ones, 1."""
    kind = rng.random()
    if kind < 0.4:
        n = 2 ** rng.randint(0, 8)
    elif kind < 0.75:
        n = 4 * _log_int(rng, 1, 64)
    else:
        n = _log_int(rng, 1, 200)
    return max(1, min(n, int(most)))


def _draw_pattern(rng, kind, most_nnz):
    if kind == "uniform":
        row = _log_int(rng, 2, 40)
        m = _log_int(rng, 700, min(500000, most_nnz // row))
        return {"m": m, "k": max(row, int(m * rng.uniform(0.6, 1.6))), "row": row}
    if kind == "stencil":
        side = min(110.0, (most_nnz / 7.0) ** (1.0 / 3.0))
        return {a: max(4, int(side * rng.uniform(0.25, 1.0))) for a in ("nx", "ny", "nz")}
    if kind == "ragged":
        mean = math.exp(rng.uniform(math.log(5.0), math.log(60.0)))
        m = _log_int(rng, 2000, min(500000, int(most_nnz / mean)))
        return {"m": m, "k": m, "mean": round(mean, 2), "sigma": round(rng.uniform(0.4, 0.9), 2),
                "band": max(1200, int(m * rng.uniform(0.02, 0.3)))}
    if kind == "graph":
        per = rng.uniform(5.0, 24.0)
        verts = _log_int(rng, 4000, min(1 << 21, int(most_nnz / per)))
        return {"scale": max(12, (verts - 1).bit_length()), "verts": verts, "edges": int(verts * per)}
    row = rng.randint(6, 40)
    m = 16 * _log_int(rng, 120, max(121, min(8192, most_nnz // (row * 256)))) + rng.choice((0, 0, 3, 11))
    return {"m": m, "k": m + rng.choice((0, 0, 5, 48)), "row": row,
            "window": min(max(24, m // 48), rng.randint(48, 600)), "fill": round(rng.uniform(0.84, 0.97), 2)}


def draw(rng):
    call = rng.choices(("spmm", "noalloc", "refresh", "epoch"), (0.66, 0.1, 0.16, 0.08))[0]
    if call == "epoch":
        verts = _log_int(rng, 3000, 262144)
        return {"call": call, "pattern": "graph", "scale": max(12, (verts - 1).bit_length()), "verts": verts,
                "edges": int(verts * rng.uniform(5.0, 16.0)), "feats": 4 * rng.randint(8, 32),
                "hidden": 4 * rng.randint(8, 32), "classes": rng.randint(7, 64)}
    if call == "noalloc":
        kind = rng.choice(("graph", "ragged", "uniform"))
        case = {"call": call, "pattern": kind, **_draw_pattern(rng, kind, 4000000)}
        return {**case, "n": _width(rng, 64)}
    if call == "refresh":
        kind = rng.choice(("graph", "graph", "ragged", "stencil", "blocks"))
        case = {"call": call, "pattern": kind, **_draw_pattern(rng, kind, 10000000)}
        return {**case, "n": _width(rng, 128), "transpose": rng.random() < 0.4}
    kind = rng.choice(("uniform", "stencil", "ragged", "graph", "graph", "blocks"))
    case = {"call": call, "pattern": kind, **_draw_pattern(rng, kind, 24000000)}
    n = _width(rng, min(256, 2.0e9 / _nnz(case)))
    return {**case, "n": n, "transpose": kind == "graph" and rng.random() < 0.5}


# --------------------------------------------------------------- patterns ---
def _shape(case):
    p = case["pattern"]
    if p == "stencil":
        m = case["nx"] * case["ny"] * case["nz"]
        return m, m
    if p == "graph":
        return case["verts"], case["verts"]
    return case["m"], case["k"]


def _nnz(case):
    """Nonzeros from the sizes alone (a graph's repeated edges are about as many as the loops added to it)."""
    p = case["pattern"]
    if p == "uniform":
        return case["m"] * case["row"]
    if p == "stencil":
        x, y, z = case["nx"], case["ny"], case["nz"]
        return 7 * x * y * z - 2 * (x * y + y * z + x * z)
    if p == "ragged":
        return int(case["m"] * case["mean"])
    if p == "graph":
        return case["edges"]
    return int((case["m"] / 16) * case["row"] * 256 * case["fill"])


def _rows_to_csr(lengths, m, k, band, g):
    """Rows of the given lengths, each row's columns distinct and ascending: entry j of a row of length L falls in
    the j-th of L equal stretches of a window of `band` columns around the row's place."""
    rowptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(lengths, 0)
    nnz = int(rowptr[-1])
    rows = torch.repeat_interleave(torch.arange(m, device=DEV), lengths, output_size=nnz)
    j = torch.arange(nnz, device=DEV) - rowptr[rows]
    length = lengths[rows]
    base = (torch.arange(m, device=DEV, dtype=torch.float64) * (k / m)).long() - band // 2
    base = base.clamp_(0, max(0, k - band))[rows]
    lo, hi = j * band // length, (j + 1) * band // length  # hi > lo: band >= length
    u = torch.rand(nnz, generator=g, device=DEV, dtype=torch.float64)
    cols = base + lo + torch.minimum((u * (hi - lo)).long(), hi - lo - 1)
    return rowptr, cols, torch.randn(nnz, generator=g, device=DEV)


def _stencil(nx, ny, nz):
    i = torch.arange(nx * ny * nz, device=DEV)
    x, y, z = i % nx, i // nx % ny, i // (nx * ny)
    steps = ((-nx * ny, z > 0), (-nx, y > 0), (-1, x > 0), (0, z >= 0), (1, x < nx - 1), (nx, y < ny - 1),
             (nx * ny, z < nz - 1))
    mask = torch.stack([ok for _, ok in steps], 1)
    cols = i[:, None] + torch.tensor([d for d, _ in steps], device=DEV)
    vals = torch.tensor([6.0 if d == 0 else -1.0 for d, _ in steps], device=DEV).expand(i.numel(), 7)
    rowptr = torch.zeros(i.numel() + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(mask.sum(1), 0)
    return rowptr, cols[mask], vals[mask].contiguous()


def _graph(scale, verts, edges, g):
    """R-MAT edges (0.57, 0.19, 0.19, 0.05) with both ends below `verts`, repeated ones merged, a loop at every
    vertex, values 1 / sqrt(d_u d_v)."""
    keys, have = [], 0
    while have < edges:
        count = min(1 << 24, int((edges - have) * 1.2) + 1024)
        r = torch.zeros(count, dtype=torch.int64, device=DEV)
        c = torch.zeros(count, dtype=torch.int64, device=DEV)
        for _ in range(scale):
            u = torch.rand(count, generator=g, device=DEV)
            low = u >= 0.76
            r = 2 * r + low
            c = 2 * c + (((u >= 0.57) & ~low) | (u >= 0.95))
        ok = (r < verts) & (c < verts)
        key = (r[ok] * verts + c[ok])[:edges - have]
        keys.append(key)
        have += key.numel()
    loops = torch.arange(verts, device=DEV) * (verts + 1)
    key = torch.unique(torch.cat(keys + [loops]))
    rows, cols = key // verts, key % verts
    deg = torch.bincount(rows, minlength=verts)
    rowptr = torch.zeros(verts + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(deg, 0)
    scale_of = deg.double().rsqrt()
    return rowptr, cols, (scale_of[rows] * scale_of[cols]).float()


def _blocks(m, k, row, window, fill, g):
    """Per block-row `row` distinct block-columns within +-window, each block filled with probability `fill`."""
    mb, kb = (m + 15) // 16, (k + 15) // 16
    span = min(2 * window, kb)
    row = min(row, span)
    j = torch.arange(row, device=DEV)
    lo, hi = j * span // row, (j + 1) * span // row
    u = torch.rand(mb, row, generator=g, device=DEV)
    base = (torch.arange(mb, device=DEV) - span // 2).clamp(0, kb - span)
    bcol = base[:, None] + lo + torch.minimum((u * (hi - lo)).long(), hi - lo - 1)
    mask = torch.rand(mb, 16, row, 16, generator=g, device=DEV) < fill
    cols = 16 * bcol[:, None, :, None] + torch.arange(16, device=DEV)
    mask &= cols < k
    mask = mask.reshape(16 * mb, row * 16)[:m]
    rowptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(mask.sum(1), 0)
    cols = cols.expand(mb, 16, row, 16).reshape(16 * mb, row * 16)[:m][mask]
    return rowptr, cols, torch.randn(cols.numel(), generator=g, device=DEV)


def _matrix(case, g):
    """(rowptr, colidx, values) on the GPU: int32, int32, float32."""
    p = case["pattern"]
    if p == "uniform":
        lengths = torch.full((case["m"],), case["row"], dtype=torch.int64, device=DEV)
        rowptr, cols, vals = _rows_to_csr(lengths, case["m"], case["k"], case["k"], g)
    elif p == "ragged":
        mu = math.log(case["mean"]) - case["sigma"] ** 2 / 2
        x = torch.randn(case["m"], generator=g, device=DEV, dtype=torch.float64)
        lengths = torch.exp(mu + case["sigma"] * x).long().clamp_(0, 480)
        lengths[::997] = 0  # a few empty rows
        rowptr, cols, vals = _rows_to_csr(lengths, case["m"], case["k"], min(case["band"], case["k"]), g)
    elif p == "stencil":
        rowptr, cols, vals = _stencil(case["nx"], case["ny"], case["nz"])
    elif p == "graph":
        rowptr, cols, vals = _graph(case["scale"], case["verts"], case["edges"], g)
    else:
        rowptr, cols, vals = _blocks(case["m"], case["k"], case["row"], case["window"], case["fill"], g)
    return rowptr.int(), cols.int(), vals


def _inputs(case, seed):
    g = torch.Generator(device=DEV).manual_seed(int(seed))
    A = _matrix(case, g)
    m, k = _shape(case)
    if case["call"] == "epoch":
        X = torch.randn(m, case["feats"], generator=g, device=DEV)
        labels = torch.randint(case["classes"], (m,), generator=g, device=DEV)
        return A, X, labels
    rows = m if case.get("transpose") else k
    return A, torch.randn(rows, case["n"], generator=g, device=DEV), None


# ------------------------------------------------------------------ calls ---
def prepare(case, seed):
    A, B, labels = _inputs(case, seed)
    m, k = _shape(case)
    nnz = A[1].numel()
    stream = torch.cuda.current_stream()
    state = {"call": case["call"], "m": m, "k": k, "nnz": nnz, "A": A, "B": B, "stream": stream}
    if case["call"] == "epoch":
        adj = torch.sparse_csr_tensor(A[0].long(), A[1].long(), A[2], (m, k))
        model = gcn.GCN2(adj, case["feats"], case["hidden"], case["classes"], DEV, seed=int(seed))
        opt = torch.optim.Adam(model.parameters(), lr=0.01)
        return {"call": "epoch", "model": model, "opt": opt, "X": B, "labels": labels}
    transpose = bool(case.get("transpose"))
    state["n"], state["transpose"] = case["n"], transpose
    state["C"] = torch.empty(k if transpose else m, case["n"], device=DEV)
    if case["call"] == "spmm":
        state["plan"] = sd.sd_plan_device(*A, m, k, nnz, case["n"], stream=stream, transpose=transpose)
        state["A"] = None  # the plan holds its own copy
    return state


def run(state):
    call = state["call"]
    if call == "epoch":
        model = state["model"]
        state["opt"].zero_grad(set_to_none=True)
        logits = model(state["X"])
        loss = torch.nn.functional.cross_entropy(logits, state["labels"])
        loss.backward()
        state["opt"].step()
        return {"loss": loss.detach(), "logits": logits.detach(), "W1": model.W1, "W2": model.W2,
                "dW1": model.W1.grad, "dW2": model.W2.grad}
    if call == "noalloc":
        sd.sd_spmm_merge_noalloc(*state["A"], state["m"], state["k"], state["nnz"], state["n"], state["B"],
                                 state["C"], stream=state["stream"])
    elif call == "refresh":
        plan = sd.sd_plan_device(*state["A"], state["m"], state["k"], state["nnz"], state["n"],
                                 stream=state["stream"], transpose=state["transpose"])
        sd.sd_spmm(plan, state["B"], state["C"], state["stream"])
        state["stream"].synchronize()  # the product is done before its plan goes
        plan.destroy()
    else:
        sd.sd_spmm(state["plan"], state["B"], state["C"], state["stream"])
    return state["C"]


def work(case):
    nnz = _nnz(case)
    m, k = _shape(case)
    csr = 8.0 * nnz + 4.0 * (m + 1)
    if case["call"] == "epoch":
        f, h, c = case["feats"], case["hidden"], case["classes"]
        # A read twice (forward, backward) at each width; X, and each layer's
        # product, activation and their gradients written and read once
        return {"bytes": 4 * csr + 4.0 * m * (2 * f + 8 * h + 8 * c),
                "flops": 4.0 * nnz * (h + c) + 4.0 * m * f * h + 6.0 * m * h * c}
    n = case["n"]
    total = {"bytes": csr + 4.0 * k * n + 4.0 * m * n, "flops": 2.0 * nnz * n}
    if case["call"] == "refresh":
        total["bytes"] += csr  # the plan's own copy
    return total


def tolerance(case):
    if case["call"] == "epoch":
        return {"rel": 2e-4, "max": 2e-2}
    return {"rel": 2e-6, "max": 1e-4}


# ------------------------------------------------------------------ exact ---
def _product64(rows, cols, vals, B, out_rows):
    out = torch.zeros(out_rows, B.shape[1], dtype=torch.float64, device=DEV)
    step = max(1, (1 << 26) // B.shape[1])
    for p in range(0, rows.numel(), step):
        at = slice(p, p + step)
        out.index_add_(0, rows[at], vals[at].double()[:, None] * B[cols[at]])
    return out


def exact(case, seed):
    (rowptr, cols, vals), B, labels = _inputs(case, seed)
    m, k = _shape(case)
    rows = torch.repeat_interleave(torch.arange(m, device=DEV), (rowptr[1:] - rowptr[:-1]).long(),
                                   output_size=cols.numel())
    cols = cols.long()
    if case["call"] != "epoch":
        if case.get("transpose"):
            return _product64(cols, rows, vals, B.double(), k)
        return _product64(rows, cols, vals, B.double(), m)

    def glorot(shape, g):
        bound = (6.0 / (shape[0] + shape[1])) ** 0.5
        return ((torch.rand(shape, generator=g, dtype=torch.float32) * 2 - 1) * bound).to(DEV).double()

    g = torch.Generator(device="cpu").manual_seed(int(seed))
    W1 = glorot((case["feats"], case["hidden"]), g)
    W2 = glorot((case["hidden"], case["classes"]), g)
    X = B.double()
    Z1 = _product64(rows, cols, vals, X @ W1, m)
    H1 = torch.relu(Z1)
    logits = _product64(rows, cols, vals, H1 @ W2, m)
    loss = torch.nn.functional.cross_entropy(logits, labels)
    G = torch.softmax(logits, 1)
    G[torch.arange(m, device=DEV), labels] -= 1.0
    G2 = _product64(cols, rows, vals, G / m, m)
    W1g, W2g = W1.clone(), W2.clone()
    W2g.grad = H1.T @ G2
    W1g.grad = X.T @ _product64(cols, rows, vals, (G2 @ W2.T) * (Z1 > 0), m)
    torch.optim.Adam([W1g, W2g], lr=0.01).step()
    return {"loss": loss, "logits": logits, "W1": W1g, "W2": W2g, "dW1": W1g.grad, "dW2": W2g.grad}
