"""Performance cases of the library's public entry points.

Each case is one piece of work that a program using the library does: a
two-phase product on a kept handle, a numeric pass that reuses the symbolic
result with new values, a chain of one-shot products, the Jacobi-fused
product, sparse addition, and batches of uneven products.  The matrices are the ones the benchmark and the tests use
(2D 5-point and 3D 27-point stencils, aggregation hierarchies, R-MAT graphs,
random rows with repeats, banded random batches), generated on the GPU: a
case's patterns are its own, their values come from the seed.  ``listed`` gives the fixed cases, ``draw`` further ones of the same
families over their whole ranges of sizes.
"""
from __future__ import annotations

import math

import torch

from paper_2103_11991_amd.spgemm import DeviceCsr, SpAdd, SpGEMM, SpGEMMBatch, spgemm

DTYPES = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # one small product on a kept handle: nothing but latency (a coarse multigrid level, a unit test)
        {"name": "lap2d_64_f64", "kind": "product", "matrix": "lap2d", "n": 64, "dtype": "f64"},
        # the smallest call: one changed-coefficient numeric pass of a small grid
        {"name": "lap2d_33_f32_reuse", "kind": "reuse", "matrix": "lap2d", "n": 33, "dtype": "f32"},
        # the headline product: A*A of a 3D 27-point stencil
        {"name": "stencil27_100_f64", "kind": "product", "matrix": "stencil27", "n": 100, "dtype": "f64"},
        # a time step with changed coefficients: the structure is known, numeric alone
        {"name": "stencil27_61_f32_reuse", "kind": "reuse", "matrix": "stencil27", "n": 61, "dtype": "f32"},
        # graph squared, power-law rows up to the widest and heaviest the library meets
        {"name": "rmat_18_f32", "kind": "product", "matrix": "rmat", "n": 1 << 18, "dtype": "f32"},
        # the same shape of graph at a size where its hub rows leave the chip partly idle
        {"name": "rmat_13_f64", "kind": "product", "matrix": "rmat", "n": 1 << 13, "dtype": "f64"},
        # rectangular matrices of scattered columns: unsorted rows, repeated entries, empty rows
        {"name": "random_rect_f64", "kind": "random", "m": 60000, "n": 45001, "k": 70003, "len_a": 24, "len_b": 24,
         "dtype": "f64"},
        # multigrid set-up: R*(A*P) down an aggregation hierarchy, one-shot products
        {"name": "galerkin_128_f64", "kind": "galerkin", "n": 128, "levels": 5, "dtype": "f64"},
        # prolongator smoothing: (I - omega D^-1 A) P, both phases
        {"name": "jacobi_128_f64", "kind": "jacobi", "n": 128, "dtype": "f64"},
        # sparse addition, the usual case: ascending rows
        {"name": "spadd_1m_sorted_f64", "kind": "spadd", "m": 1 << 20, "n": 1 << 20, "lo": 30, "hi": 30,
         "sorted": True, "dtype": "f64"},
        # sparse addition of rows as assembled: any order, repeats, empty rows
        {"name": "spadd_250k_unsorted_f32", "kind": "spadd", "m": 250007, "n": 250007, "lo": 0, "hi": 48,
         "sorted": False, "dtype": "f32"},
        # many uneven products replayed as one planned graph
        {"name": "batch_256_f64", "kind": "batch", "count": 256, "lo": 200, "hi": 50000, "dtype": "f64"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of a family of ``listed``, sizes over the family's whole range."""
    kind = rng.choice(["lap2d", "stencil27", "stencil27", "reuse", "rmat", "rmat", "random", "galerkin", "jacobi",
                       "spadd", "spadd", "batch"])
    dt = rng.choice(["f64", "f64", "f32"])
    if kind == "lap2d":
        return {"kind": "product", "matrix": "lap2d", "n": _log_int(rng, 8, 1000), "dtype": dt}
    if kind == "stencil27":
        return {"kind": "product", "matrix": "stencil27", "n": _log_int(rng, 7, 110), "dtype": dt}
    if kind == "reuse":
        return {"kind": "reuse", "matrix": rng.choice(["stencil27", "lap2d"]), "n": _log_int(rng, 9, 100), "dtype": dt}
    if kind == "rmat":
        return {"kind": "product", "matrix": "rmat", "n": _log_int(rng, 500, 140000), "dtype": dt}
    if kind == "random":
        return {"kind": "random", "m": _log_int(rng, 500, 150000), "n": _log_int(rng, 500, 150000),
                "k": _log_int(rng, 500, 150000), "len_a": rng.randint(4, 32), "len_b": rng.randint(4, 32), "dtype": dt}
    if kind == "galerkin":
        levels = rng.randint(1, 4)
        step = 1 << levels
        return {"kind": "galerkin", "n": step * rng.randint(1, 128 // step), "levels": levels, "dtype": dt}
    if kind == "jacobi":
        return {"kind": "jacobi", "n": 2 * _log_int(rng, 5, 64), "dtype": dt}
    if kind == "spadd":
        lo = rng.randint(0, 20)
        m = _log_int(rng, 1000, 1 << 20)
        return {"kind": "spadd", "m": m, "n": _log_int(rng, 1000, 1 << 20), "lo": lo, "hi": lo + rng.randint(1, 25),
                "sorted": rng.random() < 0.6, "dtype": dt}
    return {"kind": "batch", "count": _log_int(rng, 6, 300), "lo": 200, "hi": _log_int(rng, 2000, 50000), "dtype": dt}


# ------------------------------------------------------------------- matrices
def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(seed & 0x7FFFFFFF)


def _uniform(g, n, dt):
    """n values of [0, 1) in type dt, each exact in 24 bits for FP32."""
    return torch.rand(n, generator=g, device="cuda", dtype=dt)


def _from_rows(m, n, lens, cols, vals):
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=rp[1:])
    return DeviceCsr(m, n, rp.to(torch.int32), cols.to(torch.int32), vals.contiguous())


STAR2 = [(0, -1), (-1, 0), (0, 0), (1, 0), (0, 1)]
STAR3 = [(0, 0, -1), (0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
BOX3 = [(dx, dy, dz) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]


def _stencil(dims, offsets, g, dt, diagonal, spread):
    """Truncated stencil, x fastest, columns ascending: diagonal + u/2 on the
    diagonal, elsewhere -(1 + u/2), or uniform in [-1, 1) with ``spread``."""
    dims = tuple(dims) + (1,) * (3 - len(dims))
    offs = [tuple(o) + (0,) * (3 - len(o)) for o in offsets]
    nx, ny, nz = dims
    N = nx * ny * nz
    i = torch.arange(N, device="cuda")
    x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
    ok = torch.stack([(x + a >= 0) & (x + a < nx) & (y + b >= 0) & (y + b < ny) & (z + c >= 0) & (z + c < nz)
                      for a, b, c in offs], 1)
    cols = (i[:, None] + torch.tensor([a + nx * (b + ny * c) for a, b, c in offs], device="cuda")[None, :])[ok]
    diag = torch.tensor([o == (0, 0, 0) for o in offs], device="cuda")[None, :].expand(N, -1)[ok]
    u = _uniform(g, cols.numel(), dt)
    vals = torch.where(diag, diagonal + 0.5 * u, 2 * u - 1 if spread else -(1 + 0.5 * u))
    return _from_rows(N, N, ok.sum(1), cols, vals)


def _rmat(V, g, dt):
    """R-MAT on V vertices with 16 edge draws per vertex (0.57, 0.19, 0.19, 0.05): the smallest power of two that
    holds V, edges past V dropped, repeats merged; values in [0, 1)."""
    E, scale = 16 * V, max(1, (V - 1).bit_length())
    p = _rng(V)
    r = torch.zeros(E, dtype=torch.int64, device="cuda")
    c = torch.zeros(E, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        u = torch.rand(E, generator=p, device="cuda")
        rowbit = u >= 0.76
        colbit = ((u >= 0.57) & ~rowbit) | (u >= 0.95)
        r = 2 * r + rowbit
        c = 2 * c + colbit
    key = torch.unique((r * V + c)[(r < V) & (c < V)])
    return _from_rows(V, V, torch.bincount(key // V, minlength=V), key % V, _uniform(g, key.numel(), dt))


def _random_rows(m, n, lo, hi, ascending, p, g, dt):
    """Row lengths uniform in [lo, hi], columns uniform in [0, n), both drawn
    from p; ascending rows without repeats, else as drawn."""
    lens = torch.randint(lo, hi + 1, (m,), generator=p, device="cuda")
    row = torch.repeat_interleave(torch.arange(m, device="cuda"), lens)
    cols = torch.randint(0, n, (row.numel(),), generator=p, device="cuda")
    if ascending:
        key = torch.unique(row * n + cols)
        lens, cols = torch.bincount(key // n, minlength=m), key % n
    return _from_rows(m, n, lens, cols, torch.randn(cols.numel(), generator=g, device="cuda", dtype=dt))


def _aggregation(n, dt):
    """Piecewise-constant prolongator of n^3 nodes onto (n/2)^3 aggregates, and its transpose."""
    N, h = n ** 3, n // 2
    i = torch.arange(N, device="cuda")
    agg = (i % n) // 2 + h * (((i // n) % n) // 2) + h * h * ((i // (n * n)) // 2)
    one = torch.ones(N, dtype=dt, device="cuda")
    P = _from_rows(N, h ** 3, torch.ones_like(i), agg, one)
    R = _from_rows(h ** 3, N, torch.full((h ** 3,), 8, device="cuda"), torch.argsort(agg, stable=True), one.clone())
    return P, R


def _batch_sizes(case):
    """Rows and bandwidths of a batch's products: log-uniform rows, bandwidths 5..64."""
    n, bw = [], []
    for t in range(case["count"]):
        u = ((t * 0.6180339887498949) + 0.37) % 1.0
        n.append(int(round(case["lo"] * (case["hi"] / case["lo"]) ** u)))
        bw.append((5 + (t * 37) % 60, 5 + (t * 23 + 11) % 60))
    return n, bw


def _banded(n, bw, p, g, dt):
    """Square banded: 3..30 distinct ascending columns per row (drawn from p), uniform in the row's window."""
    W = 2 * bw + 1
    i = torch.arange(n, device="cuda")
    c = i[:, None] - bw + torch.arange(W, device="cuda")[None, :]
    inside = (c >= 0) & (c < n)
    want = torch.minimum(torch.randint(3, 31, (n,), generator=p, device="cuda"), inside.sum(1))
    u = torch.rand((n, W), generator=p, device="cuda").masked_fill_(~inside, 2.0)
    take = u.argsort(1).argsort(1) < want[:, None]
    cols = c[take]
    return _from_rows(n, n, want, cols, torch.randn(cols.numel(), generator=g, device="cuda", dtype=dt))


def _square(case, g):
    dt, n = DTYPES[case["dtype"]], case["n"]
    if case["matrix"] == "lap2d":
        return _stencil((n, n), STAR2, g, dt, 4.0, False)
    if case["matrix"] == "stencil27":
        return _stencil((n, n, n), BOX3, g, dt, 27.0, True)
    return _rmat(n, g, dt)


def _inputs(case, seed):
    """The case's matrices (and vectors)."""
    kind, dt = case["kind"], DTYPES[case["dtype"]]
    g, p = _rng(seed + 1), _rng(12345)  # values, patterns
    if kind == "product":
        return {"A": _square(case, g)}
    if kind == "reuse":
        A = _square(case, g)
        return {"A": A, "a": A.values + 0.25 * _uniform(g, A.nnz, dt), "b": A.values + 0.25 * _uniform(g, A.nnz, dt)}
    if kind == "random":
        return {"A": _random_rows(case["m"], case["n"], 0, case["len_a"], False, p, g, dt),
                "B": _random_rows(case["n"], case["k"], 0, case["len_b"], False, p, g, dt)}
    if kind == "galerkin":
        n = case["n"]
        return {"A": _stencil((n, n, n), STAR3, g, dt, 6.0, False),
                "PR": [_aggregation(n >> t, dt) for t in range(case["levels"])]}
    if kind == "jacobi":
        n = case["n"]
        return {"A": _stencil((n, n, n), STAR3, g, dt, 6.0, False), "P": _aggregation(n, dt)[0],
                "dinv": 1.0 / (6.0 + 0.5 * _uniform(g, n ** 3, dt))}
    if kind == "spadd":
        return {s: _random_rows(case["m"], case["n"], case["lo"], case["hi"], case["sorted"], p, g, dt) for s in "AB"}
    pairs = [(_banded(n, ba, p, g, dt), _banded(n, bb, p, g, dt)) for n, (ba, bb) in zip(*_batch_sizes(case))]
    return {"As": [p[0] for p in pairs], "Bs": [p[1] for p in pairs]}


# ------------------------------------------------------------- prepare and run
def prepare(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    x["kind"] = kind
    if kind in ("product", "reuse", "random"):
        x["op"] = SpGEMM(x["A"], x.get("B", x["A"]))
        if kind == "reuse":
            x["op"].symbolic()
    elif kind == "jacobi":
        x["op"] = SpGEMM(x["A"], x["P"])
    elif kind == "spadd":
        x["op"] = SpAdd(x["A"], x["B"])
    elif kind == "batch":
        x["op"] = SpGEMMBatch(x["As"], x["Bs"])
        x["op"].plan()
    return x


def run(x):
    kind = x["kind"]
    if kind in ("product", "random"):
        rp, _ = x["op"].symbolic()
        col, val = x["op"].numeric()
        return [rp, col, val]
    if kind == "reuse":
        return list(x["op"].numeric(a_vals=x["a"], b_vals=x["b"]))
    if kind == "galerkin":
        out, cur = [], x["A"]
        for P, R in x["PR"]:
            AP = spgemm(cur, P)
            cur = spgemm(R, AP)
            for C in (AP, cur):
                out += [C.row_ptr, C.col_idx, C.values]
        return out
    if kind == "jacobi":
        rp, _ = x["op"].symbolic()
        col, val = x["op"].numeric_jacobi(2.0 / 3.0, x["dinv"])
        return [rp, col, val]
    if kind == "spadd":
        rp, _ = x["op"].symbolic()
        col, val = x["op"].numeric(1.5, -0.75)
        return [rp, col, val]
    x["op"].run()
    return [x["op"].c_rp, x["op"].c_col, x["op"].c_val]


# ------------------------------------------------------------------------ work
def _box_count(dims, points):
    """Grid positions from which every point of ``points`` (offsets) lies in the box."""
    out = 1
    for d, n in enumerate(dims):
        at = [p[d] for p in points]
        out *= max(0, n - (max(at) - min(at)))
    return out


def _stencil_square(dims, offsets):
    """(nnz(A), products, nnz(C)) of the square of a truncated stencil matrix."""
    zero = (0,) * len(dims)
    nnz = sum(_box_count(dims, [zero, o]) for o in offsets)
    prod, sums = 0, set()
    for o in offsets:
        for p in offsets:
            s = tuple(a + b for a, b in zip(o, p))
            sums.add(s)
            prod += _box_count(dims, [zero, o, s])
    return nnz, prod, sum(_box_count(dims, [zero, s]) for s in sums)


# nnz(A), products and nnz(C) of one R-MAT square per scale
RMAT_COUNTS = {8: (2599, 87590, 26842), 10: (12094, 810540, 264005), 12: (53386, 6738667, 2406690),
               14: (228510, 53192619, 20376191), 16: (955702, 401407626, 164440464),
               18: (3940602, 2937179073, 1281758924)}


def _rmat_counts(V):
    """Their interpolation in log-log between the scales around log2(V)."""
    at = min(max(math.log2(V), 8.0), 18.0)
    lo = min(int(at) // 2 * 2, 16)
    t = (at - lo) / 2
    return tuple(a ** (1 - t) * b ** t for a, b in zip(RMAT_COUNTS[lo], RMAT_COUNTS[lo + 2]))


def _csr_bytes(m, nnz, eb):
    return 4 * (m + 1) + (4 + eb) * nnz


def work(case):
    kind, eb = case["kind"], 4 if case["dtype"] == "f32" else 8
    if kind in ("product", "reuse"):
        n = case["n"]
        if case["matrix"] == "rmat":
            rows, (nnz, prod, nc) = n, _rmat_counts(n)
        else:
            dims, offs = ((n, n), STAR2) if case["matrix"] == "lap2d" else ((n, n, n), BOX3)
            rows, (nnz, prod, nc) = n ** len(dims), _stencil_square(dims, offs)
        if kind == "reuse":  # the pattern once, two value arrays
            return {"bytes": _csr_bytes(rows, nnz, 2 * eb) + (4 + eb) * nc, "flops": 2 * prod}
        return {"bytes": _csr_bytes(rows, nnz, eb) + _csr_bytes(rows, nc, eb), "flops": 2 * prod}
    if kind == "random":
        na, nb = case["m"] * case["len_a"] / 2, case["n"] * case["len_b"] / 2
        prod = na * case["len_b"] / 2
        nc = case["m"] * case["k"] * -math.expm1(-prod / (case["m"] * case["k"]))
        return {"bytes": _csr_bytes(case["m"], na, eb) + _csr_bytes(case["n"], nb, eb) + _csr_bytes(case["m"], nc, eb),
                "flops": 2 * prod}
    if kind in ("galerkin", "jacobi"):
        total, flops, n = 0, 0, case["n"]
        for _ in range(case.get("levels", 1)):
            N, h = n ** 3, n // 2
            nnz, nap = 7 * N - 6 * n * n, 4 * N - 6 * n * n
            total += _csr_bytes(N, nnz, eb) + _csr_bytes(N, N, eb) + _csr_bytes(N, nap, eb)
            flops += 2 * nnz
            if kind == "jacobi":
                return {"bytes": total + eb * N, "flops": flops + 2 * nap}
            total += _csr_bytes(h ** 3, N, eb) + _csr_bytes(N, nap, eb) + _csr_bytes(h ** 3, 7 * h ** 3 - 6 * h * h, eb)
            flops += 2 * nap
            n = h
        return {"bytes": total, "flops": flops}
    if kind == "spadd":
        nnz = case["m"] * (case["lo"] + case["hi"]) / 2
        return {"bytes": 2 * _csr_bytes(case["m"], nnz, eb) + _csr_bytes(case["m"], 2 * nnz, eb), "flops": 4 * nnz}
    total, flops = 0, 0
    for n, (ba, bb) in zip(*_batch_sizes(case)):
        la, lb = min(16.5, 2 * ba + 1), min(16.5, 2 * bb + 1)
        width = 2 * (ba + bb) + 1
        nc = width * -math.expm1(-la * lb / width)
        total += _csr_bytes(n, n * la, eb) + _csr_bytes(n, n * lb, eb) + _csr_bytes(n, n * nc, eb)
        flops += 2 * n * la * lb
    return {"bytes": total, "flops": flops}


# ----------------------------------------------------------------------- exact
def _rows_of(A):
    rp = A.row_ptr.to(torch.int64)
    return torch.repeat_interleave(torch.arange(A.m, device="cuda"), rp[1:] - rp[:-1])


def _merge64(m, width, key, val):
    """CSR (row pointer, columns, values) of key = row * width + column with values of equal keys added."""
    key, order = torch.sort(key)
    uniq, inverse = torch.unique_consecutive(key, return_inverse=True)
    out = torch.zeros(uniq.numel(), dtype=torch.float64, device="cuda").index_add_(0, inverse, val[order])
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(uniq // width, minlength=m), 0, out=rp[1:])
    return rp, uniq % width, out


def _product64(A, a, B, b, most=1 << 27):
    """C = A*B with values a, b in 64 bits: all products, sorted by row and column, in slices of A's rows."""
    arp, brp = A.row_ptr.to(torch.int64), B.row_ptr.to(torch.int64)
    acol, bcol = A.col_idx.to(torch.int64), B.col_idx.to(torch.int64)
    blen = brp[1:] - brp[:-1]
    upto = torch.zeros(A.nnz + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(blen[acol], 0, out=upto[1:])
    done = upto[arp]
    rows, width = _rows_of(A), max(B.n, 1)
    a, b = a.to(torch.float64), b.to(torch.float64)
    parts, r0 = [], 0
    while r0 < A.m:
        r1 = int(torch.searchsorted(done, done[r0] + most, right=True).item()) - 1
        r1 = min(max(r1, r0 + 1), A.m)
        e0, e1 = int(arp[r0]), int(arp[r1])
        e = torch.arange(e0, e1, device="cuda")
        e = torch.repeat_interleave(e, upto[e + 1] - upto[e])
        q = brp[acol[e]] + (torch.arange(e.numel(), device="cuda") + upto[e0] - upto[e])
        parts.append(_merge64(r1 - r0, width, (rows[e] - r0) * width + bcol[q], a[e] * b[q]))
        r0 = r1
    rp = [torch.zeros(1, dtype=torch.int64, device="cuda")]
    for p in parts:
        rp.append(p[0][1:] + rp[-1][-1])
    empty = torch.zeros(0, dtype=torch.int64, device="cuda")
    return (torch.cat(rp), torch.cat([p[1] for p in parts] or [empty]),
            torch.cat([p[2] for p in parts] or [empty.to(torch.float64)]))


def exact(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("product", "random"):
        B = x.get("B", x["A"])
        return list(_product64(x["A"], x["A"].values, B, B.values))
    if kind == "reuse":
        return list(_product64(x["A"], x["a"], x["A"], x["b"])[1:])
    if kind == "galerkin":
        out, cur = [], x["A"]
        for P, R in x["PR"]:
            for left, right in ((None, P), (R, None)):
                L, M = left or cur, right or cur
                cur = DeviceCsr(L.m, M.n, *_product64(L, L.values, M, M.values))
                out += [cur.row_ptr, cur.col_idx, cur.values]
        return out
    if kind == "jacobi":
        A, P = x["A"], x["P"]
        scale = -(2.0 / 3.0) * x["dinv"].to(torch.float64)[_rows_of(A)]
        rp, col, val = _product64(A, A.values.to(torch.float64) * scale, P, P.values)
        C = DeviceCsr(A.m, P.n, rp, col, val)
        key = torch.cat([_rows_of(C) * P.n + col, _rows_of(P) * P.n + P.col_idx.to(torch.int64)])
        return list(_merge64(A.m, P.n, key, torch.cat([val, P.values.to(torch.float64)])))
    if kind == "spadd":
        A, B = x["A"], x["B"]
        key = torch.cat([_rows_of(M) * M.n + M.col_idx.to(torch.int64) for M in (A, B)])
        return list(_merge64(A.m, A.n, key, torch.cat([1.5 * A.values.double(), -0.75 * B.values.double()])))
    parts = [_product64(A, A.values, B, B.values) for A, B in zip(x["As"], x["Bs"])]
    rp = [torch.zeros(1, dtype=torch.int64, device="cuda")]
    for p in parts:
        rp.append(p[0][1:] + rp[-1][-1])
    return [torch.cat(rp), torch.cat([p[1] for p in parts]), torch.cat([p[2] for p in parts])]
