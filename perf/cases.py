"""Timed workloads of the sparse product library, one pass each.

Every case is one call (or the few calls that belong together) as a program
that uses the library makes them: whole products, the numeric phase alone on
a structure that is kept, batches of multigrid products, the adjoint, an
autograd step, triangle counting and a product under an HBM budget. Matrices
are the library's own workload families (grid stencils, smoothed-aggregation
prolongators, Poisson-random rows, R-MAT graphs), generated on the GPU from a
seed; structures depend on the case alone (so that every seed gives outputs of
one shape), values on the seed. The graphs of triangle counting, whose output
has the shape of the vertices, are drawn from the seed.

listed()      the cases that stand for the range
draw(rng)     one more case of the same ranges
prepare       inputs, structures, plans and handles a program keeps
run           one pass, returning every output
work          bytes and floating-point operations of one pass
exact         the floating outputs in 64 bits from plain torch operations
"""
import itertools
import random

import numpy as np
import torch

import paper_1804_00695_amd as mls

DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases

def listed():
    return [
        # coarse multigrid level: a product of a few thousand rows, launch and synchronisation bound
        {"name": "product_laplace2d_64", "kind": "product", "matrix": "laplace2d", "n": 64},
        # general rectangular product of ragged random rows, still small
        {"name": "product_poisson_3000", "kind": "product", "matrix": "poisson", "rows": 3000, "inner": 2000,
         "cols": 2500, "row_a": 5.0, "row_b": 7.0},
        # fine-level operator squared: the largest in-memory product
        {"name": "product_stencil27_128", "kind": "product", "matrix": "stencil27", "n": 128},
        # power-law graph squared: hub rows past every on-chip table
        {"name": "product_rmat_16", "kind": "product", "matrix": "rmat", "scale": 16, "edge_factor": 8},
        # restriction times operator, values changed and structure kept (81 entries per row, long rows of B)
        {"name": "numeric_elasticity_RA", "kind": "numeric", "matrix": "elasticity3d", "n": 48, "product": "RA"},
        # setup of several small multigrid hierarchies at once: A*P, then R*(A*P), structures and values
        {"name": "galerkin_batch_20", "kind": "galerkin", "count": 20, "lo": 16, "hi": 64},
        # the same setup repeated with new values on kept structures (captured plan)
        {"name": "galerkin_replay_32", "kind": "replay", "count": 32, "lo": 16, "hi": 64},
        # gradient of a large random product, fastest mode
        {"name": "adjoint_random_1M", "kind": "adjoint", "rows": 1000000, "row_a": 8.0, "row_b": 8.0,
         "deterministic": False},
        # the same repeatable bit for bit
        {"name": "adjoint_fixed_order_200k", "kind": "adjoint", "rows": 200003, "row_a": 8.0, "row_b": 8.0,
         "deterministic": True},
        # a training step of moderate size: forward values and both gradients through autograd
        {"name": "autograd_random_20k", "kind": "autograd", "rows": 20011, "row_a": 6.0, "row_b": 6.0},
        # triangle count of a power-law graph
        {"name": "triangles_rmat_18", "kind": "triangles", "scale": 18, "edge_factor": 16},
        # the numeric phase from pinned host memory under an HBM budget
        {"name": "chunked_stencil27_64", "kind": "chunked", "n": 64, "budget_mb": 128, "nbuf": 2, "min_parts": 4,
         "in_place": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["product", "product", "product", "numeric", "galerkin", "replay", "adjoint", "adjoint",
                       "autograd", "triangles", "chunked"])
    if kind == "product":
        matrix = rng.choice(["laplace2d", "stencil27", "poisson", "rmat"])
        if matrix == "laplace2d":
            return {"kind": kind, "matrix": matrix, "n": _log_int(rng, 20, 1000)}
        if matrix == "stencil27":
            return {"kind": kind, "matrix": matrix, "n": _log_int(rng, 9, 127)}
        if matrix == "rmat":
            return {"kind": kind, "matrix": matrix, "scale": rng.randint(10, 15),
                    "edge_factor": rng.randint(4, 12)}
        return {"kind": kind, "matrix": matrix, "rows": _log_int(rng, 300, 500000),
                "inner": _log_int(rng, 300, 500000), "cols": _log_int(rng, 300, 500000),
                "row_a": round(rng.uniform(2.0, 12.0), 2), "row_b": round(rng.uniform(2.0, 12.0), 2)}
    if kind == "numeric":
        matrix, lo, hi = rng.choice([("laplace3d", 20, 120), ("bigstar2d", 100, 1200), ("brick3d", 16, 90),
                                     ("elasticity3d", 8, 48)])
        return {"kind": kind, "matrix": matrix, "n": _log_int(rng, lo, hi), "product": rng.choice(["RA", "AP"])}
    if kind in ("galerkin", "replay"):
        lo = rng.randint(6, 30)
        return {"kind": kind, "count": rng.randint(2, 20 if kind == "galerkin" else 32), "lo": lo,
                "hi": lo + rng.randint(1, 34)}
    if kind == "adjoint":
        return {"kind": kind, "rows": _log_int(rng, 500, 600000), "row_a": round(rng.uniform(2.0, 10.0), 2),
                "row_b": round(rng.uniform(2.0, 10.0), 2), "deterministic": rng.random() < 0.4}
    if kind == "autograd":
        return {"kind": kind, "rows": _log_int(rng, 500, 300000), "row_a": round(rng.uniform(2.0, 10.0), 2),
                "row_b": round(rng.uniform(2.0, 10.0), 2)}
    if kind == "triangles":
        return {"kind": kind, "scale": rng.randint(10, 18), "edge_factor": rng.randint(4, 16)}
    return {"kind": kind, "n": rng.randint(24, 64), "budget_mb": rng.choice([64, 96, 128, 256, 1024]),
            "nbuf": rng.randint(1, 4), "min_parts": rng.randint(1, 4), "in_place": rng.random() < 0.3}


# ---------------------------------------------------------------------------
# matrices (DeviceCsr), structures from sizes, values from the generator g

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _row_ptr(counts):
    rp = torch.zeros(counts.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(counts, 0, out=rp[1:])
    return rp.to(torch.int32)


OFFSETS = {
    "laplace2d": (2, [(0, 0), (-1, 0), (1, 0), (0, -1), (0, 1)], 1),
    "laplace3d": (3, [(0, 0, 0), (-1, 0, 0), (1, 0, 0), (0, -1, 0), (0, 1, 0), (0, 0, -1), (0, 0, 1)], 1),
    "bigstar2d": (2, [(0, 0), (-1, 0), (1, 0), (0, -1), (0, 1), (-2, 0), (2, 0), (0, -2), (0, 2),
                      (-1, -1), (-1, 1), (1, -1), (1, 1)], 1),
    "stencil27": (3, list(itertools.product((-1, 0, 1), repeat=3)), 1),
    "brick3d": (3, list(itertools.product((-1, 0, 1), repeat=3)), 1),
    "elasticity3d": (3, list(itertools.product((-1, 0, 1), repeat=3)), 3),
}


def _coords(n, dim):
    i = torch.arange(n ** dim, device=DEV)
    return i, [(i // n ** (dim - 1 - d)) % n for d in range(dim)]


def _masked_rows(valid, col, val, nrows, ncols):
    """CSR of the valid entries of dense per-row candidate lists (columns ascending along a row)."""
    return mls.DeviceCsr(nrows, ncols, _row_ptr(valid.sum(1)), col[valid].to(torch.int32), val[valid])


def operator(matrix, n, g):
    """Stencil operator on an n^dim grid: off-diagonal values -(1 + U(-0.1, 0.1)), a dominant diagonal."""
    dim, offs, dof = OFFSETS[matrix]
    offs = sorted(offs)
    i, xs = _coords(n, dim)
    N = n ** dim
    valid = torch.ones(N, len(offs), dtype=torch.bool, device=DEV)
    flat = torch.zeros(len(offs), dtype=torch.int64)
    for o, off in enumerate(offs):
        for d, od in enumerate(off):
            c = xs[d] + od
            valid[:, o] &= (c >= 0) & (c < n)
            flat[o] += od * n ** (dim - 1 - d)
    nbr = i[:, None] + flat.to(DEV)[None, :]
    a = torch.arange(dof, device=DEV)
    shape = (N, dof, len(offs), dof)
    valid = valid[:, None, :, None].expand(shape).reshape(N * dof, -1)
    col = (nbr[:, None, :, None] * dof + a).expand(shape).reshape(N * dof, -1)
    val = -1.0 - 0.1 * (2.0 * torch.rand(col.shape, generator=g, device=DEV, dtype=torch.float64) - 1.0)
    row = torch.arange(N * dof, device=DEV)
    val = torch.where(col == row[:, None], float(len(offs) * dof) - 0.5, val)
    return _masked_rows(valid, col, val, N * dof, N * dof)


def prolongator(matrix, n, g):
    """Smoothed aggregation over 2 nodes per dimension: up to 1 + dim entries per row, weights varied by 5 %."""
    dim, _, dof = OFFSETS[matrix]
    nc = (n + 1) // 2
    i, xs = _coords(n, dim)
    N, Nc = n ** dim, nc ** dim
    agg = sum((xs[d] // 2) * nc ** (dim - 1 - d) for d in range(dim))
    same = sum(((x % 2 == 1) | ((x % 2 == 0) & (x + 1 < n))).to(torch.float64) for x in xs)
    minus = [((x >= 1) & (x % 2 == 0), -nc ** (dim - 1 - d)) for d, x in enumerate(xs)]
    plus = [((x + 1 < n) & (x % 2 == 1), nc ** (dim - 1 - d)) for d, x in enumerate(xs)]
    cands = minus + [(torch.ones(N, dtype=torch.bool, device=DEV), 0)] + plus[::-1]
    valid = torch.stack([ok for ok, _ in cands], 1)
    col = torch.stack([agg + off for _, off in cands], 1)
    w = torch.full(col.shape, 1.0 / (3 * dim), dtype=torch.float64, device=DEV)
    w[:, dim] = (dim + same) / (3 * dim)
    valid = valid.repeat_interleave(dof, 0)
    col = (col[:, None, :] * dof + torch.arange(dof, device=DEV)[None, :, None]).reshape(N * dof, -1)
    w = w.repeat_interleave(dof, 0)
    w = w * (1.0 + 0.05 * (2.0 * torch.rand(w.shape, generator=g, device=DEV, dtype=torch.float64) - 1.0))
    return _masked_rows(valid, col, w, N * dof, Nc * dof)


def transposed(M):
    order = torch.argsort(M.col_idx, stable=True)
    rows = _rows_of(M)
    return mls.DeviceCsr(M.ncols, M.nrows, _row_ptr(torch.bincount(M.col_idx, minlength=M.ncols)),
                         rows[order].to(torch.int32), M.values[order])


def poisson(nrows, ncols, lam, gs, g):
    """Rows of Poisson(lam) distinct uniform columns drawn from gs, N(0, 1) values from g."""
    k = torch.poisson(torch.full((nrows,), float(lam), device=DEV), generator=gs).to(torch.int64).clamp_(max=ncols)
    rows = torch.repeat_interleave(torch.arange(nrows, device=DEV), k)
    key = rows * ncols + torch.randint(0, ncols, rows.shape, generator=gs, device=DEV)
    key = torch.unique(key)   # a column drawn twice in a row is kept once
    return _from_keys(key, nrows, ncols, torch.randn(key.shape, generator=g, device=DEV, dtype=torch.float64))


def rmat_keys(scale, edge_factor, g):
    """Symmetric R-MAT graph (.57, .19, .19, .05) without self loops: sorted keys row * 2^scale + column."""
    m, n = edge_factor << scale, 1 << scale
    u = torch.zeros(m, dtype=torch.int64, device=DEV)
    v = torch.zeros(m, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        r = torch.rand(m, generator=g, device=DEV)
        u = (u << 1) | (r >= 0.76)
        v = (v << 1) | (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    u, v = u[u != v], v[u != v]
    return torch.unique(torch.cat([u * n + v, v * n + u]))


def lower_by_degree(key, n):
    """Pattern of the strict lower triangle after relabelling by descending degree (ties by ascending id)."""
    u, v = key // n, key % n
    perm = torch.argsort(torch.bincount(u, minlength=n), descending=True, stable=True)
    new = torch.empty_like(perm)
    new[perm] = torch.arange(n, device=DEV)
    u, v = new[u], new[v]
    return _from_keys(torch.sort((u * n + v)[v < u])[0], n, n, None)


def _from_keys(key, nrows, ncols, values):
    return mls.DeviceCsr(nrows, ncols, _row_ptr(torch.bincount(key // ncols, minlength=nrows)),
                         (key % ncols).to(torch.int32), values)


def _rows_of(M):
    return torch.repeat_interleave(torch.arange(M.nrows, device=DEV), torch.diff(M.row_ptr).to(torch.int64))


def _pinned(M):
    def pin(t):
        h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
        h.copy_(t)
        return h
    return mls.HostCsr(M.nrows, M.ncols, pin(M.row_ptr), pin(M.col_idx), pin(M.values))


def _grid_sizes(case):
    r = random.Random(4)   # the sizes belong to the case, the values to the seed
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["count"])]


def _factors(case, seed):
    """(A, B) of a case of one product."""
    g, gs = _gen(seed), _gen(5)
    m = case.get("matrix")
    if case["kind"] == "numeric":
        A, P = operator(m, case["n"], g), prolongator(m, case["n"], g)
        return (transposed(P), A) if case["product"] == "RA" else (A, P)
    if case["kind"] in ("adjoint", "autograd"):
        n = case["rows"]
        return poisson(n, n, case["row_a"], gs, g), poisson(n, n, case["row_b"], gs, g)
    if m == "poisson":
        return (poisson(case["rows"], case["inner"], case["row_a"], gs, g),
                poisson(case["inner"], case["cols"], case["row_b"], gs, g))
    if m == "rmat":
        key = rmat_keys(case["scale"], case["edge_factor"], gs)
        n = 1 << case["scale"]
        A = _from_keys(key, n, n, torch.randn(key.shape, generator=g, device=DEV, dtype=torch.float64))
        return A, A
    A = operator(m or "stencil27", case["n"], g)
    return A, A


def _hierarchies(case, seed):
    g = _gen(seed)
    As, Ps, Rs = [], [], []
    for n in _grid_sizes(case):
        As.append(operator("laplace3d", n, g))
        Ps.append(prolongator("laplace3d", n, g))
        Rs.append(transposed(Ps[-1]))
    return As, Ps, Rs


def _weights(C, seed):
    return torch.randn(C.nnz, generator=_gen(seed + 1), device=DEV, dtype=torch.float64)


# ---------------------------------------------------------------------------
# prepare and run

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("galerkin", "replay"):
        As, Ps, Rs = _hierarchies(case, seed)
        s = {"kind": kind, "As": As, "Ps": Ps, "Rs": Rs}
        if kind == "replay":
            s["APs"] = mls.batch_symbolic(As, Ps)
            s["Acs"] = mls.batch_symbolic(Rs, s["APs"])
            s["plans"] = mls.BatchPlan(As, Ps, s["APs"]), mls.BatchPlan(Rs, s["APs"], s["Acs"])
        return s
    if kind == "triangles":
        n = 1 << case["scale"]
        return {"kind": kind, "L": lower_by_degree(rmat_keys(case["scale"], case["edge_factor"], _gen(seed)), n)}
    A, B = _factors(case, seed)
    s = {"kind": kind, "A": A, "B": B}
    if kind == "product":
        return s
    C = mls.symbolic(A, B)
    s["C"] = C
    if kind == "adjoint":
        s["W"] = mls.DeviceCsr(C.nrows, C.ncols, C.row_ptr, C.col_idx, _weights(C, seed))
        s["deterministic"] = case["deterministic"]
    elif kind == "autograd":
        s["av"], s["bv"] = A.values.clone().requires_grad_(), B.values.clone().requires_grad_()
        s["w"] = _weights(C, seed)
    elif kind == "chunked":
        h = _pinned(A)
        s["A"] = s["B"] = h
        s["C"] = _pinned(C)
        rp = h.row_ptr.numpy()
        s["plan"] = mls.chunked_plan(rp, rp, A.ncols, s["C"].row_ptr.numpy(), case["budget_mb"] << 20,
                                     nbuf=case["nbuf"], min_parts=case["min_parts"], knl=case["in_place"])
        s["streams"] = mls.ChunkStreams()
    return s


def run(s):
    kind = s["kind"]
    if kind == "product":
        C = mls.spgemm(s["A"], s["B"])
        return C.row_ptr, C.col_idx, C.values
    if kind == "numeric":
        return mls.numeric(s["A"], s["B"], s["C"]).values
    if kind == "galerkin":
        APs = mls.batch_symbolic(s["As"], s["Ps"])
        mls.batch_numeric(s["As"], s["Ps"], APs)
        Acs = mls.batch_symbolic(s["Rs"], APs)
        mls.batch_numeric(s["Rs"], APs, Acs)
        return [(C.row_ptr, C.col_idx, C.values) for C in Acs]
    if kind == "replay":
        for plan in s["plans"]:
            plan.run()
        return [C.values for C in s["APs"]], [C.values for C in s["Acs"]]
    if kind == "adjoint":
        return mls.backward(s["A"], s["B"], s["W"], deterministic=s["deterministic"])
    if kind == "autograd":
        cv = mls.SpGEMMFn.apply(s["av"], s["bv"], s["A"], s["B"], s["C"])
        ga, gb = torch.autograd.grad(cv, (s["av"], s["bv"]), s["w"])
        return cv.detach(), ga, gb
    if kind == "triangles":
        return mls.triangle_count(s["L"])
    return mls.numeric_chunked(s["A"], s["B"], s["C"], s["plan"], streams=s["streams"]).values


# ---------------------------------------------------------------------------
# what a pass cannot do without

def _bytes(M, values=True):
    return 4 * (M.nrows + 1) + (12 if values else 4) * M.nnz


def _entry_work(A, B):
    return torch.diff(B.row_ptr).to(torch.int64)[A.col_idx.to(torch.int64)]


def work(case):
    kind = case["kind"]
    if kind in ("galerkin", "replay"):
        # the intermediate A*P is an output of the replay alone
        As, Ps, Rs = _hierarchies(case, 0)
        APs = mls.batch_symbolic(As, Ps, with_values=False)
        Acs = mls.batch_symbolic(Rs, APs, with_values=False)
        nbytes = sum(_bytes(M) for M in As + Ps + Rs + Acs + (APs if kind == "replay" else []))
        madds = sum(int(_entry_work(X, Y).sum()) for X, Y in list(zip(As, Ps)) + list(zip(Rs, APs)))
        return {"bytes": nbytes, "flops": 2 * madds}
    if kind == "triangles":
        L = lower_by_degree(rmat_keys(case["scale"], case["edge_factor"], _gen(0)), 1 << case["scale"])
        return {"bytes": _bytes(L, values=False) + 8 * L.nrows, "flops": 0}
    A, B = _factors(case, 0)
    C = mls.symbolic(A, B, with_values=False)
    madds = int(_entry_work(A, B).sum())
    nbytes = _bytes(A) + (_bytes(B) if B is not A else 0) + _bytes(C)
    if kind == "adjoint":
        return {"bytes": nbytes + 8 * (A.nnz + B.nnz), "flops": 4 * madds}
    if kind == "autograd":
        return {"bytes": nbytes + 8 * C.nnz + 8 * (A.nnz + B.nnz), "flops": 6 * madds}
    return {"bytes": nbytes, "flops": 2 * madds}


# ---------------------------------------------------------------------------
# the same in 64 bits with plain torch operations

def _row_blocks(A, B, most=1 << 25):
    """Row ranges of A of about `most` multiply-adds each."""
    per_entry = torch.zeros(A.nnz + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(_entry_work(A, B), 0, out=per_entry[1:])
    upto = per_entry[A.row_ptr.to(torch.int64)].cpu().numpy()
    r = 0
    while r < A.nrows:
        e = max(r + 1, int(np.searchsorted(upto, upto[r] + most, side="right")) - 1)
        yield r, min(e, A.nrows)
        r = e


def _triples(A, B, r0, r1):
    """Entries (of A, of B) of every multiply-add of rows [r0, r1), and the keys of the outputs they go to."""
    p0, p1 = int(A.row_ptr[r0]), int(A.row_ptr[r1])
    k = A.col_idx[p0:p1].to(torch.int64)
    first = B.row_ptr.to(torch.int64)[k]
    cnt = B.row_ptr.to(torch.int64)[k + 1] - first
    ea = torch.repeat_interleave(torch.arange(p1 - p0, device=DEV), cnt)
    eb = (first - (torch.cumsum(cnt, 0) - cnt))[ea] + torch.arange(ea.numel(), device=DEV)
    lens = torch.diff(A.row_ptr[r0:r1 + 1]).to(torch.int64)
    rows = torch.repeat_interleave(torch.arange(r0, r1, device=DEV), lens)
    return ea + p0, eb, rows[ea] * B.ncols + B.col_idx[eb]


def _product(A, B):
    keys, vals = [], []
    for r0, r1 in _row_blocks(A, B):
        ea, eb, key = _triples(A, B, r0, r1)
        u, inv = torch.unique(key, return_inverse=True)
        vals.append(torch.zeros(u.numel(), dtype=torch.float64, device=DEV)
                    .index_add_(0, inv, A.values[ea] * B.values[eb]))
        keys.append(u)
    return _from_keys(torch.cat(keys), A.nrows, B.ncols, torch.cat(vals))


def _adjoint(A, B, C, w):
    dA = torch.zeros(A.nnz, dtype=torch.float64, device=DEV)
    dB = torch.zeros(B.nnz, dtype=torch.float64, device=DEV)
    ckey = _rows_of(C) * C.ncols + C.col_idx
    for r0, r1 in _row_blocks(A, B):
        ea, eb, key = _triples(A, B, r0, r1)
        wv = w[torch.searchsorted(ckey, key)]
        dA.index_add_(0, ea, wv * B.values[eb])
        dB.index_add_(0, eb, wv * A.values[ea])
    return dA, dB


def exact(case, seed):
    kind = case["kind"]
    if kind == "triangles":
        return None   # whole numbers only
    if kind in ("galerkin", "replay"):
        As, Ps, Rs = _hierarchies(case, seed)
        APs = [_product(A, P) for A, P in zip(As, Ps)]
        Acs = [_product(R, X) for R, X in zip(Rs, APs)]
        if kind == "galerkin":
            return [(None, None, C.values) for C in Acs]
        return [C.values for C in APs], [C.values for C in Acs]
    A, B = _factors(case, seed)
    C = _product(A, B)
    if kind == "product":
        return None, None, C.values
    if kind in ("adjoint", "autograd"):
        dA, dB = _adjoint(A, B, C, _weights(C, seed))
        return (dA, dB) if kind == "adjoint" else (C.values, dA, dB)
    return C.values
