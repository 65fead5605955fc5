"""Timed cases of the sparse product C = A*B.

The cases cover what a program uses the library for: whole products in one
call, one row panel of a product too large for memory, a product cut into
panels, and a product repeated for new values on kept patterns; irregular
matrices (R-MAT, the sizes and parameters of the benchmark workloads and of
the A*B grid), regular ones (banded, grid stencils, uniform random), square
and rectangular; fp64 and fp32 values, int32 and int64 columns.
"""
from __future__ import annotations

import math

import torch

from paper_2607_22866_amd import gmagnus as g

GRAPH500 = (0.57, 0.19, 0.19)
SKEWED = (0.60, 0.17, 0.17)


def listed():
    return [
        # the smallest product: a graph of 4096 vertices, where launches and host reads count
        {"name": "rmat12_square", "kind": "rmat", "scale": 12, "a_ef": 8, "b_ef": 0, "skewed": False},
        # a mid-size graph squared in one call (one multisplit level)
        {"name": "rmat17_square", "kind": "rmat", "scale": 17, "a_ef": 16, "b_ef": 0, "skewed": False},
        # the headline workload: one row panel of the scale-22 square
        {"name": "rmat22_panel", "kind": "panel", "scale": 22, "a_ef": 16, "b_ef": 0, "skewed": False,
         "products": 2_000_000_000, "at": 0.4},
        # the sparser, more skewed scale-23 square: wide first-level chunks
        {"name": "rmat23_panel", "kind": "panel", "scale": 23, "a_ef": 8, "b_ef": 0, "skewed": True,
         "products": 1_500_000_000, "at": 0.7},
        # fp32 values: a row panel of a scale-18 square
        {"name": "rmat18_f32_panel", "kind": "panel", "scale": 18, "a_ef": 16, "b_ef": 0, "skewed": False,
         "products": 1_000_000_000, "at": 0.3, "value": "float32"},
        # the A*B grid: distinct matrices of different densities, the rows split into panels first
        {"name": "rmat17_pair_panels", "kind": "pair", "scale": 17, "a_ef": 32, "b_ef": 8, "skewed": False,
         "products": 400_000_000},
        # new values on kept patterns (two multisplit levels): the values-only re-run
        {"name": "rmat19_pair_values", "kind": "values", "scale": 19, "a_ef": 4, "b_ef": 4, "skewed": False},
        # banded matrix of the benchmark: every row's columns fit a narrow window
        {"name": "banded20_square", "kind": "banded", "n": 1 << 20, "half": 13},
        # 27-point stencil on an odd-sized grid: regular rows with wide column spans and many repeats
        {"name": "stencil27_square", "kind": "stencil", "nx": 103, "ny": 99, "nz": 101, "points": 27},
        # uniform random matrix of the benchmark: hardly any repeats, C as large as the products
        {"name": "er22_square", "kind": "er", "m": 1 << 22, "k": 1 << 22, "n": 1 << 22, "a_d": 16, "b_d": 16},
        # denser uniform rows with 64-bit columns, an odd size
        {"name": "er_d40_i64", "kind": "er", "m": 250_007, "k": 250_007, "n": 250_007, "a_d": 40, "b_d": 40,
         "index": "int64"},
        # rectangular product with few products per row
        {"name": "rect_few", "kind": "er", "m": 400_003, "k": 60_013, "n": 300_007, "a_d": 6, "b_d": 9},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rmat_products(scale, a_ef, b_ef, skewed):
    """Expected products of two R-MAT matrices, repeated edges counted."""
    a, b, c = SKEWED if skewed else GRAPH500
    d = 1.0 - a - b - c
    return 4.0 ** scale * a_ef * b_ef * ((a + c) * (a + b) + (b + d) * (c + d)) ** scale


def draw(rng):
    kind = rng.choice(["rmat", "rmat", "panel", "panel", "pair", "values", "banded", "stencil", "er", "er"])
    case = {"kind": kind}
    if kind in ("rmat", "pair", "values"):
        limit = {"rmat": 1.0e9, "pair": 1.0e9, "values": 4.0e8}[kind]
        while True:
            scale = rng.randint(10, 17) if kind == "rmat" else rng.randint(13, 18)
            a_ef = rng.randint(4, 32)
            b_ef = rng.randint(4, 16) if kind != "rmat" or rng.random() < 0.3 else 0
            skewed = rng.random() < 0.3
            est = _rmat_products(scale, a_ef, b_ef or a_ef, skewed)
            if est <= limit:
                break
        case.update(scale=scale, a_ef=a_ef, b_ef=b_ef, skewed=skewed)
        if kind == "pair":
            case["products"] = max(100_000, int(est / rng.uniform(1.5, 8.0)))
    elif kind == "panel":
        case.update(scale=rng.randint(18, 22), a_ef=rng.randint(6, 16), b_ef=0, skewed=rng.random() < 0.3,
                    products=_log_int(rng, 5e7, 1e9), at=round(rng.random(), 3))
    elif kind == "banded":
        case.update(n=_log_int(rng, 1 << 13, 1 << 20), half=rng.randint(1, 26))
    elif kind == "stencil":
        case.update(nx=rng.randint(20, 100), ny=rng.randint(20, 100), nz=rng.randint(20, 100),
                    points=rng.choice([7, 27]))
    else:
        while True:
            m, k, n = (_log_int(rng, 1 << 13, 1 << 21) for _ in range(3))
            a_d, b_d = rng.randint(2, 48), rng.randint(2, 48)
            if rng.random() < 0.5:
                k = n = m
            if m * a_d * b_d <= 5e8 and a_d <= k and b_d <= n:
                break
        case.update(m=m, k=k, n=n, a_d=a_d, b_d=b_d)
    if rng.random() < 0.3:
        case["value"] = "float32"
    # (fp32 R-MAT products of more than 2^18 columns run with 64-bit columns only)
    if rng.random() < 0.2 or (case.get("value") == "float32" and case.get("scale", 0) > 18):
        case["index"] = "int64"
    return case


# ------------------------------------------------------------------- inputs
def _types(case):
    return getattr(torch, case.get("index", "int32")), getattr(torch, case.get("value", "float64"))


def _csr(case, n_rows, n_cols, keys):
    """CSR pattern from the sorted distinct keys row * n_cols + column."""
    it, vt = _types(case)
    rows = torch.div(keys, n_cols, rounding_mode="floor")
    cols = (keys - rows * n_cols).to(it)
    rp = torch.zeros(n_rows + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n_rows), 0)
    return g.DeviceCSR(n_rows, n_cols, rp, cols, torch.empty(0, dtype=vt, device="cuda"))


def _values(gen, n, vt, positive):
    v = torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)
    return (v if positive else v.mul_(2.0).sub_(1.0)).to(vt)


def _rmat(case, gen, ef):
    """R-MAT edges, one uniform draw per bit and edge; repeated edges are one entry."""
    a, b, c = SKEWED if case["skewed"] else GRAPH500
    scale = case["scale"]
    n = 1 << scale
    key_r = torch.zeros(n * ef, dtype=torch.int64, device="cuda")
    key_c = torch.zeros_like(key_r)
    for _ in range(scale):
        u = torch.rand(n * ef, device="cuda", generator=gen)
        low = u >= a + b
        right = ((u >= a) & ~low) | (u >= a + b + c)
        key_r.mul_(2).add_(low)
        key_c.mul_(2).add_(right)
    keys = torch.unique(key_r.mul_(n).add_(key_c))
    return _csr(case, n, n, keys)


def _uniform(case, gen, n_rows, n_cols, d):
    """About d distinct uniform columns in every row."""
    cols = torch.randint(0, n_cols, (n_rows, d), device="cuda", generator=gen)
    cols.add_(torch.arange(n_rows, device="cuda").mul_(n_cols)[:, None])
    return _csr(case, n_rows, n_cols, torch.unique(cols.flatten()))


def _banded(case):
    n, half = case["n"], case["half"]
    i = torch.arange(n, device="cuda")[:, None]
    j = i + torch.arange(-half, half + 1, device="cuda")[None, :]
    ok = (j >= 0) & (j < n)
    return _csr(case, n, n, (i * n + j)[ok])


def _stencil(case):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n = nx * ny * nz
    i = torch.arange(n, device="cuda")
    x, y, z = i % nx, torch.div(i, nx, rounding_mode="floor") % ny, torch.div(i, nx * ny, rounding_mode="floor")
    keys, oks = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if case["points"] == 7 and abs(dx) + abs(dy) + abs(dz) > 1:
                    continue
                oks.append((x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz >= 0) & (z + dz < nz))
                keys.append(i * n + i + dx + dy * nx + dz * nx * ny)
    return _csr(case, n, n, torch.stack(keys, 1)[torch.stack(oks, 1)])


def _matrices(case, gen):
    if case["kind"] == "banded":
        A = _banded(case)
        return A, A
    if case["kind"] == "stencil":
        A = _stencil(case)
        return A, A
    if case["kind"] == "er":
        A = _uniform(case, gen, case["m"], case["k"], case["a_d"])
        if case["m"] == case["k"] == case["n"] and case["a_d"] == case["b_d"]:
            return A, A
        return A, _uniform(case, gen, case["k"], case["n"], case["b_d"])
    A = _rmat(case, gen, case["a_ef"])
    return A, (_rmat(case, gen, case["b_ef"]) if case["b_ef"] else A)


def prepare(case, seed):
    # The patterns belong to the case, so that C has the same size for every
    # seed; the seed gives the values.
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2607)
    A, B = _matrices(case, gen)
    gen.manual_seed(seed)
    positive = "scale" in case
    A.val = _values(gen, A.nnz, A.value_dtype, positive)
    if B is not A:
        B.val = _values(gen, B.nnz, B.value_dtype, positive)
    state = {"kind": case["kind"], "A": A, "B": B, "rows": (0, A.n_rows)}
    if case["kind"] == "panel":
        bounds = g.split_panels(A, B, case["products"])
        p = int(case["at"] * (len(bounds) - 2))
        state["rows"] = (bounds[p], bounds[p + 1])
    elif case["kind"] == "pair":
        state["products"] = case["products"]
    elif case["kind"] == "values":
        plan = g.Plan(A, B, flags=g.FLAG_KEEP_PATTERN)
        state["row_ptr"], _ = plan.symbolic()
        plan.numeric()
        state["plan"] = plan
        state["a_val"] = _values(gen, A.nnz, A.value_dtype, True)
        state["b_val"] = state["a_val"] if B is A else _values(gen, B.nnz, B.value_dtype, True)
    return state


def run(state):
    A, B = state["A"], state["B"]
    if state["kind"] == "panel":
        return g.spgemm(A, B, row_begin=state["rows"][0], row_end=state["rows"][1])
    if state["kind"] == "pair":
        bounds = g.split_panels(A, B, state["products"])
        return [g.spgemm(A, B, row_begin=a, row_end=b) for a, b in zip(bounds[:-1], bounds[1:])]
    if state["kind"] == "values":
        state["plan"].update_values(state["a_val"], state["b_val"])
        return (state["row_ptr"],) + tuple(state["plan"].numeric())
    return g.spgemm(A, B)


# ------------------------------------------------------------ work, reference
def work(case):
    """Inputs read once, C written once; two operations a product."""
    s = prepare(case, 1)
    A, B = s["A"], s["B"]
    r0, r1 = s["rows"]
    ip = _row_products(A, B)[r0:r1]
    with g.Plan(A, B, row_begin=r0, row_end=r1) as p:
        nnz_c = p.symbolic()[1]
    entry = A.col.element_size() + A.val.element_size()
    a_nnz = int(A.row_ptr[r1] - A.row_ptr[r0])
    byts = 8 * (r1 - r0 + 1) + entry * a_nnz + 8 * (r1 - r0 + 1) + entry * nnz_c
    if B is not A or case["kind"] == "panel":
        byts += 8 * (B.n_rows + 1) + entry * B.nnz
    return {"bytes": float(byts), "flops": 2.0 * float(ip.sum())}


def _row_products(A, B):
    lens = (B.row_ptr[1:] - B.row_ptr[:-1])[A.col.long()]
    pre = torch.zeros(A.nnz + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=pre[1:])
    return pre[A.row_ptr[1:]] - pre[A.row_ptr[:-1]]


def tolerance(case):
    # another order of the sums (up to 6e-7 in fp32 and 1.1e-15 in fp64 against 64-bit sums of sorted
    # products, of up to some thousands of terms); structure exact
    return {"rel": 2e-6, "max": 1e-5} if case.get("value") == "float32" else {"rel": 4e-15, "max": 2e-14}


def _product(A, B, a_val, b_val, r0, r1):
    """Rows [r0, r1) of A*B: every product formed in 64 bits, sorted by (row, column), runs summed."""
    ip = _row_products(A, B)[r0:r1]
    pre = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(ip, 0)])
    cuts, r = [0], 0
    pre_h = pre.cpu()
    while r < r1 - r0:
        r = max(int(torch.searchsorted(pre_h, pre_h[r] + 250_000_000, right=True)) - 1, r + 1)
        r = min(r, r1 - r0)
        cuts.append(r)
    cols, vals, counts = [], [], []
    for a, b in zip(cuts[:-1], cuts[1:]):
        e0, e1 = int(A.row_ptr[r0 + a]), int(A.row_ptr[r0 + b])
        row = torch.repeat_interleave(torch.arange(b - a, device="cuda"),
                                      A.row_ptr[r0 + a + 1:r0 + b + 1] - A.row_ptr[r0 + a:r0 + b])
        k = A.col[e0:e1].long()
        lens = B.row_ptr[k + 1] - B.row_ptr[k]
        first = torch.cumsum(lens, 0) - lens
        e = torch.repeat_interleave(torch.arange(e1 - e0, device="cuda"), lens)
        src = torch.arange(e.numel(), device="cuda").add_((B.row_ptr[k] - first)[e])
        prod = b_val.double()[src].mul_(a_val[e0:e1].double()[e])
        key = B.col[src].long().add_(row[e] * B.n_cols)
        del src, e
        key, order = torch.sort(key)
        prod = prod[order]
        del order
        key, run_len = torch.unique_consecutive(key, return_counts=True)
        run = torch.repeat_interleave(torch.arange(key.numel(), device="cuda"), run_len)
        vals.append(torch.zeros(key.numel(), dtype=torch.float64, device="cuda").index_add_(0, run, prod))
        rows = torch.div(key, B.n_cols, rounding_mode="floor")
        cols.append((key - rows * B.n_cols).to(A.col.dtype))
        counts.append(torch.bincount(rows, minlength=b - a))
        del key, run, run_len, prod, rows
    rp = torch.zeros(r1 - r0 + 1, dtype=torch.int64, device="cuda")
    if counts:
        rp[1:] = torch.cumsum(torch.cat(counts), 0)
    empty = torch.zeros(0, dtype=torch.float64, device="cuda")
    return rp, torch.cat(cols) if cols else empty.to(A.col.dtype), torch.cat(vals) if vals else empty


def exact(case, seed):
    s = prepare(case, seed)
    A, B = s["A"], s["B"]
    if s["kind"] == "values":
        s["plan"].close()
        return _product(A, B, s["a_val"], s["b_val"], 0, A.n_rows)
    if s["kind"] == "pair":
        bounds = g.split_panels(A, B, s["products"])
        return [_product(A, B, A.val, B.val, a, b) for a, b in zip(bounds[:-1], bounds[1:])]
    return _product(A, B, A.val, B.val, *s["rows"])
