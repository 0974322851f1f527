"""Performance cases of the SpGEMM library: the work its users have it do, through the public entry points.

Every case is one pass of one of the library's paths:

  product   C = A B, symbolic and numeric phase (square A A of a graph, or a rectangular A B)
  layers    the c windowed layer products of one split product, then their merge
  merge     the merge of c partial products that are there already
  summa     one process's Sparse SUMMA stages on a hypersparse share of a larger square product
  galerkin  a batch of (R^T A) R products whose structure stays and whose values may change, replayed
  amg       one level of an AMG setup: MIS-2 aggregation, R and R^T, R^T A and (R^T A) R
  learned   the product with predicted row sizes

Matrices are R-MAT graphs (G500, SSCA), uniform ones (ER), or 7-point grid operators, all made on the GPU.  A case
fixes a graph up to the order of its vertices; the seed relabels them (another structure with as many entries in every
result) and draws the values.  `exact` computes the same results by expanding and sorting every scalar product in plain torch.
"""

import math
import random

import torch

import paper_1510_00844_amd as spg
from paper_1510_00844_amd import learned as sizer

# R-MAT quadrant probabilities
CLASSES = {
    "g500": (0.57, 0.19, 0.19, 0.05),
    "ssca": (0.6, 0.4 / 3, 0.4 / 3, 0.4 / 3),
    "er": (0.25, 0.25, 0.25, 0.25),
}
DTYPE = {"f64": torch.float64, "i64": torch.int64, "bool": torch.uint8}
DEV = "cuda"


def listed():
    return [
        # the smallest call: 65,536 scalar products, so launches and read-backs are what it costs
        dict(name="er12_f64", path="product", cls="er", m=4096, k=4096, n=4096, per_row=4, square=True, sr="f64"),
        # rectangular, odd sizes, structure and truth values only (reachability between two vertex sets)
        dict(name="rect_bool", path="product", cls="g500", m=30011, k=47777, n=25013, per_row=16, square=False,
             sr="bool"),
        # counting paths of length two in a sparser power-law graph
        dict(name="ssca16_i64", path="product", cls="ssca", m=1 << 16, k=1 << 16, n=1 << 16, per_row=8, square=True,
             sr="i64"),
        # the headline workload: squaring a G500 graph of scale 16
        dict(name="g500_16_f64", path="product", cls="g500", m=1 << 16, k=1 << 16, n=1 << 16, per_row=16, square=True,
             sr="f64"),
        # two independent uniform matrices of scale 18: every row alike, hardly any equal columns
        dict(name="er18_f64", path="product", cls="er", m=1 << 18, k=1 << 18, n=1 << 18, per_row=16, square=False,
             sr="f64"),
        # the largest configuration: squaring a G500 graph of scale 19 (billions of scalar products)
        dict(name="g500_19_f64", path="product", cls="g500", m=1 << 19, k=1 << 19, n=1 << 19, per_row=16, square=True,
             sr="f64"),
        # the split product of one process column: four layer products and their merge
        dict(name="layers4_er18_f64", path="layers", cls="er", m=1 << 18, k=1 << 18, n=1 << 18, per_row=16, layers=4,
             sr="f64"),
        # the merge alone, of the sixteen layers that arrive from a deep third grid dimension
        dict(name="merge16_er18_f64", path="merge", cls="er", m=1 << 18, k=1 << 18, n=1 << 18, per_row=16, layers=16,
             sr="f64"),
        # one process of a 16 x 16 x 4 grid squaring a G500 graph of scale 20, stage blocks of 4096
        dict(name="summa20_f64", path="summa", cls="g500", scale=20, per_row=16, grid=16, layers=4, block=4096,
             sr="f64"),
        # the coarse operators of 64 grid problems at once, new values on known structures
        dict(name="galerkin64_f64", path="galerkin", count=64, nmin=16, nmax=64, sr="f64"),
        # one level of an AMG setup on a single odd-sized grid
        dict(name="amg75_f64", path="amg", grid=75, sr="f64"),
        # the product with predicted row sizes on a G500 graph
        dict(name="learned15_f64", path="learned", cls="g500", m=1 << 15, k=1 << 15, n=1 << 15, per_row=16,
             square=True, sr="f64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: any path, sizes spread over their logarithm, odd ones among them."""
    path = rng.choice(["product", "product", "product", "layers", "merge", "summa", "galerkin", "amg", "learned"])
    sr = rng.choice(["f64", "f64", "f64", "i64", "bool"])
    if path in ("product", "learned"):
        cls = "g500" if path == "learned" else rng.choice(["g500", "ssca", "er"])
        n = _log_int(rng, 2000, 1 << (16 if path == "learned" else 18))
        per_row = rng.randint(3, 16)
        if path == "learned" or rng.random() < 0.6:
            return dict(path=path, cls=cls, m=n, k=n, n=n, per_row=per_row, square=True, sr=sr)
        return dict(path=path, cls=cls, m=_log_int(rng, n / 3, n), k=n, n=_log_int(rng, n / 3, n), per_row=per_row,
                    square=False, sr=sr)
    if path in ("layers", "merge"):
        n = _log_int(rng, 4000, 1 << 18)
        return dict(path=path, cls=rng.choice(["er", "er", "ssca"]) if n <= 1 << 16 else "er", m=n, k=n, n=n,
                    per_row=rng.randint(4, 16), layers=_log_int(rng, 2, 16), sr=sr)
    if path == "summa":
        scale = rng.randint(16, 20)
        return dict(path=path, cls="g500", scale=scale, per_row=rng.randint(8, 16), grid=16, layers=4,
                    block=(1 << (scale - 2)) // 16 // rng.choice([1, 2, 4, 8, 16]), sr=sr)
    if path == "galerkin":
        nmin = rng.randint(8, 24)
        return dict(path=path, count=_log_int(rng, 4, 64), nmin=nmin, nmax=nmin + rng.randint(4, 40), sr=sr)
    return dict(path=path, grid=_log_int(rng, 16, 100), sr=sr)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & ((1 << 62) - 1))
    return g


def _values(count, sr, g):
    if sr == "f64":
        return torch.rand(count, dtype=torch.float64, device=DEV, generator=g)
    if sr == "i64":
        return torch.randint(1, 4, (count,), dtype=torch.int64, device=DEV, generator=g)
    return torch.ones(count, dtype=torch.uint8, device=DEV)


def _row_ptr(rows, m):
    """Row pointers of sorted row indices."""
    return torch.searchsorted(rows, torch.arange(m + 1, device=DEV))


def _csr(m, n, key, sr, g):
    """Canonical CSR of the sorted distinct keys row * n + column, with new values."""
    rows = torch.div(key, n, rounding_mode="floor")
    return spg.DeviceCSR(m, n, _row_ptr(rows, m), (key - rows * n).to(torch.int32), _values(key.numel(), sr, g))


def _rmat(m, n, edges, cls, salt, same):
    """Distinct (row, column) pairs of an m x n R-MAT graph whose vertices are shuffled; `same`: rows and columns by one
    permutation.  The same graph on every call with the same arguments."""
    g = _gen(1000003 * edges + 101 * m + 11 * n + salt)
    a, b, c, _ = CLASSES[cls]
    s = max(1, (max(m, n) - 1).bit_length())
    rows = torch.zeros(edges, dtype=torch.int64, device=DEV)
    cols = torch.zeros(edges, dtype=torch.int64, device=DEV)
    for _ in range(s):
        u = torch.rand(edges, device=DEV, generator=g)
        rows = rows * 2 + (u >= a + b)
        cols = cols * 2 + (((u >= a) & (u < a + b)) | (u >= a + b + c))
    p = torch.randperm(1 << s, device=DEV, generator=g)
    q = p if same else torch.randperm(1 << s, device=DEV, generator=g)
    key = torch.unique(((p[rows] * m) >> s) * n + ((q[cols] * n) >> s))
    rows = torch.div(key, n, rounding_mode="floor")
    return rows, key - rows * n


def _order(n, g):
    return torch.randperm(n, device=DEV, generator=g)


def _placed(m, n, rows, cols, sr, g):
    return _csr(m, n, (rows * n + cols).sort().values, sr, g)


def _operands(case, seed):
    g = _gen(seed)
    m, k, n, e = case["m"], case["k"], case["n"], case["per_row"]
    square = case.get("square", False)
    p, q, r = _order(m, g), _order(k, g), _order(n, g)
    rows, cols = _rmat(m, k, e * m, case["cls"], 1, square)
    if square:
        A = _placed(m, m, p[rows], p[cols], case["sr"], g)
        return A, A
    A = _placed(m, k, p[rows], q[cols], case["sr"], g)
    rows, cols = _rmat(k, n, e * k, case["cls"], 2, False)
    return A, _placed(k, n, q[rows], r[cols], case["sr"], g)


def _bounds(case):
    k, c = case["k"], case["layers"]
    return [((l * k) // c, ((l + 1) * k) // c) for l in range(c)]


def _window(A, lo, hi):
    """A's entries with column in [lo, hi), as a matrix of the same shape."""
    rows = torch.repeat_interleave(torch.arange(A.nrows, device=DEV), A.row_ptr.diff())
    keep = (A.col >= lo) & (A.col < hi)
    return spg.DeviceCSR(A.nrows, A.ncols, _row_ptr(rows[keep], A.nrows), A.col[keep],
                         None if A.val is None else A.val[keep])


def _summa_share(case, seed):
    """Process (0, 1, 1)'s rows of A and columns of B over its layer's inner indices."""
    g = _gen(seed)
    n = 1 << case["scale"]
    mb, kb = n // case["grid"], n // case["layers"]
    rows, cols = _rmat(n, n, case["per_row"] * n, case["cls"], 1, True)
    p, q, r = _order(mb, g), _order(kb, g), _order(mb, g)
    a = (rows < mb) & (cols >= kb) & (cols < 2 * kb)
    b = (rows >= kb) & (rows < 2 * kb) & (cols >= mb) & (cols < 2 * mb)
    A = _placed(mb, kb, p[rows[a]], q[cols[a] - kb], case["sr"], g)
    B = _placed(kb, mb, q[rows[b] - kb], r[cols[b] - mb], case["sr"], g)
    return A, B


def _compress(A):
    """The kept (non-empty) rows of A."""
    ids = torch.nonzero(A.row_ptr.diff()).flatten()
    return spg.DeviceDCSR(A.nrows, A.ncols, ids.to(torch.int32), torch.cat([A.row_ptr[ids], A.row_ptr[-1:]]), A.col,
                          A.val)


def _poisson(N, sr, g):
    """7-point operator on an N^3 grid (Dirichlet) with varying coefficients, -1 (i64: whole numbers) on the faces."""
    idx = torch.arange(N ** 3, device=DEV)
    x, y, z = idx % N, torch.div(idx, N, rounding_mode="floor") % N, torch.div(idx, N * N, rounding_mode="floor")
    keys = [idx * N ** 3 + idx]
    for d, (dx, dy, dz) in ((-1, (-1, 0, 0)), (1, (1, 0, 0)), (-N, (0, -1, 0)), (N, (0, 1, 0)), (-N * N, (0, 0, -1)),
                            (N * N, (0, 0, 1))):
        ok = ((x + dx >= 0) & (x + dx < N) & (y + dy >= 0) & (y + dy < N) & (z + dz >= 0) & (z + dz < N))
        keys.append(idx[ok] * N ** 3 + idx[ok] + d)
    A = _csr(N ** 3, N ** 3, torch.cat(keys).sort().values, sr, g)
    if sr != "bool":  # diagonal positive, faces negative, coefficients of about 6 and 1
        rows = torch.repeat_interleave(idx, A.row_ptr.diff())
        one = A.val if sr == "i64" else A.val + 0.5
        A.val = torch.where(A.col == rows, 6 * one, -one)
    return A


def _blocks(N):
    """The aggregate of every point: 2 x 2 x 2 blocks."""
    M = (N + 1) // 2
    idx = torch.arange(N ** 3, device=DEV)
    x, y, z = idx % N, torch.div(idx, N, rounding_mode="floor") % N, torch.div(idx, N * N, rounding_mode="floor")
    return x // 2 + M * (y // 2 + M * (z // 2)), M ** 3


def _grid_sizes(case):
    r = random.Random(5)
    return [r.randint(case["nmin"], case["nmax"]) for _ in range(case["count"])]


def _restriction(N, sr):
    agg, M = _blocks(N)
    n = N ** 3
    one = torch.ones(n, dtype=DTYPE[sr], device=DEV)
    R = spg.DeviceCSR(n, M, torch.arange(n + 1, device=DEV), agg.to(torch.int32), one)
    rows, order = torch.sort(agg, stable=True)
    return R, spg.DeviceCSR(M, n, _row_ptr(rows, M), order.to(torch.int32), one)


def _batch(case, seed):
    g = _gen(seed)
    sizes = _grid_sizes(case)
    A = [_poisson(N, case["sr"], g) for N in sizes]
    R, RT = zip(*(_restriction(N, case["sr"]) for N in sizes))
    return sizes, list(RT), A, list(R)


# ---------------------------------------------------------------------------
# the paths
# ---------------------------------------------------------------------------
def prepare(case, seed):
    path, st = case["path"], {"path": case["path"], "sr": case["sr"], "plan": spg.Plan()}
    if path in ("product", "layers", "learned"):
        st["A"], st["B"] = _operands(case, seed)
        if path == "layers":
            st["bounds"] = _bounds(case)
        if path == "learned":
            st["params"] = sizer.load()
    elif path == "merge":
        A, B = _operands(case, seed)
        st["layers"] = [_plain_product(_window(A, lo, hi), B, case["sr"]) for lo, hi in _bounds(case)]
    elif path == "summa":
        A, B = _summa_share(case, seed)
        st["A"], st["B"], st["stages"], st["block"] = _compress(A), B, case["grid"], case["block"]
    elif path == "galerkin":
        _, st["RT"], st["A"], st["R"] = _batch(case, seed)
    elif path == "amg":
        st["A"], st["seed"] = _poisson(case["grid"], case["sr"], _gen(seed)), 5
    else:
        raise ValueError(path)
    return st


def _parts(C):
    return C.row_ptr, C.col, C.val


def run(st):
    path, plan, sr = st["path"], st["plan"], st["sr"]
    if path == "product":
        return _parts(spg.spgemm(plan, sr, st["A"], st["B"]))
    if path == "layers":
        parts = [spg.spgemm(plan, sr, st["A"], st["B"], lo, hi) for lo, hi in st["bounds"]]
        return _parts(spg.spgemm_merge_layers(plan, sr, parts))
    if path == "merge":
        return _parts(spg.spgemm_merge_layers(plan, sr, st["layers"]))
    if path == "summa":
        C, kept = spg.spgemm_summa_local(plan, sr, st["A"], st["B"], st["stages"], st["block"])
        return C.row_ids, C.row_ptr, C.col, C.val, kept
    if path == "galerkin":
        C = spg.spgemm_galerkin_batched(plan, sr, st["RT"], st["A"], st["R"]).fetch(plan)
        # the instances lie back to back in one buffer each of row pointers, columns and values
        nnz, rows = sum(c.nnz for c in C), sum(c.nrows + 1 for c in C)
        return (C[0].row_ptr.as_strided((rows,), (1,)), C[0].col.as_strided((nnz,), (1,)),
                C[0].val.as_strided((nnz,), (1,)))
    if path == "amg":
        in_mis, agg, n_agg, _ = spg.spg_mis2_aggregate(plan, st["A"], st["seed"])
        R, RT = spg.spg_restriction(plan, sr, agg, n_agg)
        C = spg.spgemm(plan, sr, spg.spgemm(plan, sr, RT, st["A"]), R)
        return (in_mis, agg, RT.row_ptr, RT.col) + _parts(C)
    C, _ = spg.spgemm_learned(plan, sr, st["A"], st["B"], st["params"])
    return _parts(C)


# ---------------------------------------------------------------------------
# what a pass needs, and its exact result, in plain torch
# ---------------------------------------------------------------------------
def _lengths(A, B):
    """nnz(B(k,:)) of every stored A(i,k), and the row of every stored A(i,k)."""
    rows = torch.repeat_interleave(torch.arange(A.nrows, device=DEV), A.row_ptr.diff())
    return B.row_ptr.diff()[A.col.long()], rows


def _expand(A, B, lens, rows, p0, p1, sr):
    """Keys row * n + column and values of the products of A's entries [p0, p1)."""
    ln = lens[p0:p1]
    ent = torch.repeat_interleave(torch.arange(p1 - p0, device=DEV), ln)
    first = torch.cumsum(ln, 0) - ln
    q = (B.row_ptr[A.col[p0:p1].long()] - first)[ent] + torch.arange(ent.numel(), device=DEV)
    key = rows[p0:p1][ent] * B.ncols + B.col[q].long()
    val = None if sr is None else A.val[p0:p1][ent] * B.val[q]
    return key, val


def _plain_product(A, B, sr, most=1 << 26):
    """A B by expanding every product, a run of whole rows at a time, and adding those with the same place."""
    lens, rows = _lengths(A, B)
    zero = torch.zeros(1, dtype=torch.int64, device=DEV)
    upto = torch.cat([zero, torch.cumsum(lens, 0)])[A.row_ptr].cpu().numpy()
    rp = A.row_ptr.cpu().numpy()
    keys, vals, i = [], [], 0
    while i < A.nrows:
        j = max(i + 1, int(upto.searchsorted(upto[i] + most, side="right")) - 1)
        if rp[j] > rp[i]:
            key, val = _expand(A, B, lens, rows, rp[i], rp[j], sr)
            u, inv = torch.unique(key, return_inverse=True)
            if sr == "bool":
                v = torch.zeros(u.numel(), dtype=torch.int32, device=DEV).index_add_(0, inv, val.int())
                v = (v > 0).to(torch.uint8)
            else:
                v = torch.zeros(u.numel(), dtype=val.dtype, device=DEV).index_add_(0, inv, val)
            keys.append(u)
            vals.append(v)
        i = j
    key = torch.cat(keys) if keys else zero[:0]
    val = torch.cat(vals) if vals else torch.zeros(0, dtype=DTYPE[sr], device=DEV)
    r = torch.div(key, B.ncols, rounding_mode="floor")
    return spg.DeviceCSR(A.nrows, B.ncols, _row_ptr(r, A.nrows), (key - r * B.ncols).to(torch.int32), val)


def _products(A, B):
    return int(_lengths(A, B)[0].sum()) if A.nnz else 0


def _outputs(A, B, most=1 << 25):
    """nnz(A B), from a sample of rows where there are many products."""
    total = _products(A, B)
    step = max(1, -(-total // most))
    lens, rows = _lengths(A, B)
    keep = rows % step == 0
    sub = spg.DeviceCSR(A.nrows, A.ncols, A.row_ptr, A.col[keep], None)
    key, _ = _expand(sub, B, lens[keep], rows[keep], 0, int(keep.sum()), None)
    return min(total, torch.unique(key).numel() * total // max(1, key.numel()))


def exact(case, seed):
    path, sr = case["path"], case["sr"]
    if path in ("product", "layers", "merge", "learned"):
        A, B = _operands(case, seed)
        return None if _products(A, B) > 1 << 30 else _parts(_plain_product(A, B, sr))
    if path == "summa":
        A, B = _summa_share(case, seed)
        C = _compress(_plain_product(A, B, sr))
        return C.row_ids, C.row_ptr, C.col, C.val, None
    if path == "galerkin":
        sizes, _, A, _ = _batch(case, seed)
        rps, cols, vals = [], [], []
        for N, a in zip(sizes, A):
            agg, M = _blocks(N)
            rows = torch.repeat_interleave(torch.arange(a.nrows, device=DEV), a.row_ptr.diff())
            u, inv = torch.unique(agg[rows] * M + agg[a.col.long()], return_inverse=True)
            v = torch.zeros(u.numel(), dtype=torch.int32 if sr == "bool" else a.val.dtype, device=DEV)
            v.index_add_(0, inv, a.val.to(v.dtype))
            r = torch.div(u, M, rounding_mode="floor")
            rps.append(_row_ptr(r, M))
            cols.append((u - r * M).to(torch.int32))
            vals.append((v > 0).to(torch.uint8) if sr == "bool" else v)
        return torch.cat(rps), torch.cat(cols), torch.cat(vals)
    return None  # amg: the aggregates are the library's own


def _bytes(sr, *matrices):
    """Stored size of matrices given as (rows, entries)."""
    w = 4 + {"f64": 8, "i64": 8, "bool": 1}[sr]
    return float(sum(8 * (rows + 1) + w * nnz for rows, nnz in matrices))


def work(case):
    """Each operand read once and each result written once; a multiplication and an addition per scalar product (an
    addition per entry that a merge or an aggregation reads)."""
    path, sr = case["path"], case["sr"]
    if path in ("product", "layers", "learned", "merge"):
        A, B = _operands(case, 0)
        flops, out = _products(A, B), _outputs(A, B)
        if path == "merge":  # the layers hold nearly as many entries as there are products
            return {"bytes": _bytes(sr, (case["m"], out)) + _bytes(sr, *[(case["m"], flops / case["layers"])] * case["layers"]),
                    "flops": float(flops)}
        own = [(A.nrows, A.nnz)] if A is B else [(A.nrows, A.nnz), (B.nrows, B.nnz)]
        return {"bytes": _bytes(sr, *own, (case["m"], out)), "flops": 2.0 * flops}
    if path == "summa":
        A, B = _summa_share(case, 0)
        kept = int((A.row_ptr.diff() > 0).sum())
        return {"bytes": _bytes(sr, (kept, A.nnz), (B.nrows, B.nnz), (kept, _outputs(A, B))),
                "flops": 2.0 * _products(A, B)}
    total, flops = 0.0, 0.0
    for N in _grid_sizes(case) if path == "galerkin" else [case["grid"]]:
        a, M = 7 * N ** 3 - 6 * N * N, ((N + 1) // 2) ** 3
        if path == "galerkin":
            total += _bytes(sr, (N ** 3, a), (N ** 3, N ** 3), (M, N ** 3), (M, 7 * M))
        else:  # about 20 points an aggregate; A read, the aggregates, R, R^T and a small C written
            M = N ** 3 // 20 + 1
            total += _bytes(sr, (N ** 3, a), (N ** 3, N ** 3), (M, N ** 3), (M, 15 * M)) + 5.0 * N ** 3
        flops += 4.0 * a
    return {"bytes": total, "flops": flops}
