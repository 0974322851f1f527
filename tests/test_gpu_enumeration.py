"""The product enumeration of the workgroup kernels at its edges: rows of one
A entry more or less than a batch holds (448 in workgroups of 512 threads, 960
in those of 1024), batches of empty and one-entry B rows (more than 64 segments
in a step of 64 products), and long B rows beside them, through the symbolic
bitmap, the whole-row rank, the rank-chunk (one and several chunks, one and
several items per row, both gather pipelines) and the hash kernels.  INT64 is
exact; FP64 uses the suite's per-entry bound."""

import numpy as np
import pytest
import torch

import oracle
import paper_1510_00844_amd as spg
import synth
from gpu_util import check_full_vs_oracle, to_dev
from synth.gen import canonical_from_coo

pytestmark = pytest.mark.gpu

K = 3000
COUNTS = [2, 63, 64, 65, 447, 448, 449, 500, 896, 897, 959, 960, 961, 1921, 2600]


def operands(lens, n, seed):
    """A with rows of COUNTS entries (all B rows they can reach), B with rows
    of the given length pattern."""
    rng = np.random.default_rng(seed)
    blen = {"short": rng.choice([0, 0, 1, 2], K), "ones": np.ones(K, np.int64),
            "mixed": np.where(rng.random(K) < 0.02, rng.integers(200, 900, K), rng.integers(0, 4, K)),
            "even": np.full(K, 16)}[lens]
    rows, cols = [], []
    for r, c in enumerate(COUNTS):
        rows.append(np.full(c, r))
        cols.append(rng.choice(K, c, replace=False))
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    A = canonical_from_coo(len(COUNTS), K, rows, cols, rng.uniform(-1, 1, rows.size), dup="first")
    br = np.repeat(np.arange(K), blen)
    bc = np.concatenate([rng.choice(n, c, replace=False) for c in blen])
    return A, canonical_from_coo(K, n, br, bc, rng.uniform(-1, 1, br.size), dup="first")


OPTS = {
    "default": {},
    "rank1024": dict(rank_block=1024),
    "chunks": dict(rank_max_nnz=1, chunk_min_nnz=1, dense_chunk_cols=2048),
    "chunks_pipelined": dict(rank_max_nnz=1, chunk_min_nnz=1, dense_chunk_cols=2048, gather_pipeline=2),
    "one_chunk_items": dict(rank_max_nnz=1, chunk_min_nnz=1, chunk_group=1),
    "many_words": dict(rank_max_nnz=1, chunk_min_nnz=1, chunk_group=256, dense_chunk_cols=16384),
    "per_thread": dict(gather_map=2, sym_gather_map=2),
    "eight": dict(unroll=8, sym_unroll=8, chunk_unroll=8, rank_max_nnz=1, chunk_min_nnz=1),
}


@pytest.mark.parametrize("opts", list(OPTS))
@pytest.mark.parametrize("lens,n", [("short", 1500), ("ones", 3000), ("mixed", 20011), ("even", 40000), ("mixed", 200003)])
def test_enumeration_edges(opts, lens, n):
    print("case enumeration", opts, lens, n, flush=True)
    A, B = operands(lens, n, seed=3)
    plan = spg.Plan(**OPTS[opts])
    for sr in ("f64", "i64"):
        if sr == "i64":
            A.val, B.val = np.rint(A.val * 9).astype(np.int64), np.rint(B.val * 9).astype(np.int64)
        a, b = to_dev(A, sr), to_dev(B, sr)
        for _ in range(2):  # the second call takes the counts of the first
            check_full_vs_oracle(spg.spgemm(plan, sr, a, b), A, B, sr)
    plan.close()


@pytest.mark.parametrize("opts", ["default", "chunks"])
def test_enumeration_special_values(opts):
    """Infinities and NaN reach exactly the entries whose terms hold them."""
    A, B = operands("mixed", 20011, seed=4)
    rng = np.random.default_rng(0)
    B.val[rng.choice(B.nnz, 40, replace=False)] = np.inf
    B.val[rng.choice(B.nnz, 40, replace=False)] = np.nan
    plan = spg.Plan(**OPTS[opts])
    C = spg.spgemm(plan, "f64", to_dev(A), to_dev(B))
    D = torch.zeros(B.nrows, B.ncols, dtype=torch.float64)
    rows = np.repeat(np.arange(B.nrows), np.diff(B.row_ptr))
    D[rows, B.col.astype(np.int64)] = torch.from_numpy(B.val)
    rp, col, val = C.to_numpy()
    for i in range(A.nrows):
        ks = A.col[A.row_ptr[i]:A.row_ptr[i + 1]].astype(np.int64)
        js = torch.from_numpy(col[rp[i]:rp[i + 1]].astype(np.int64))
        t = D[torch.from_numpy(ks)][:, js] * torch.from_numpy(A.val[A.row_ptr[i]:A.row_ptr[i + 1]])[:, None]
        ref = t.sum(0)
        got = torch.from_numpy(val[rp[i]:rp[i + 1]])
        assert torch.equal(torch.isnan(got), torch.isnan(ref))
        assert torch.equal(torch.isinf(got), torch.isinf(ref))
    plan.close()


@pytest.mark.parametrize("sizes", [[64, 65, 1, 63], [4096, 2, 65], [1000] * 3 + [1] * 70 + [129], [1]])
def test_restriction_row_lengths(sizes):
    """R^T rows around the register sort's 64 and up to the LDS sort's 4096."""
    rng = np.random.default_rng(1)
    agg = rng.permutation(np.repeat(np.arange(len(sizes)), sizes)).astype(np.int32)
    plan = spg.Plan()
    R, RT = spg.spg_restriction(plan, "i64", torch.from_numpy(agg).cuda(), len(sizes))
    order = np.argsort(agg, kind="stable")
    assert np.array_equal(RT.row_ptr.cpu().numpy(), np.concatenate([[0], np.cumsum(sizes)]))
    assert np.array_equal(RT.col.cpu().numpy(), order)
    assert np.array_equal(R.col.cpu().numpy(), agg)
    with pytest.raises(spg.SpgError):
        spg.spg_restriction(plan, "i64", torch.zeros(4097, dtype=torch.int32, device="cuda"), 1)
    plan.close()


@pytest.mark.parametrize("window", [None, (100, 5900)])
@pytest.mark.parametrize("reps", [1, 90])
def test_row_analysis_lengths(window, reps):
    """Rows around the lengths where the row analysis changes hands (16 lanes
    per row to 128 entries, a wave to 2048, the workgroup above), the row
    pointers and lists of more than one 1024-row tile, and the bin statistics."""
    k, n = 6000, 700
    counts = np.tile([0, 1, 15, 16, 17, 32, 33, 127, 128, 129, 300, 2047, 2048, 2049, 5000], reps)
    rng = np.random.default_rng(2)
    order = np.argsort(rng.random((64, k)), axis=1)
    rows = np.repeat(np.arange(counts.size), counts)
    cols = np.concatenate([order[i % 64, :c] for i, c in enumerate(counts)])
    A = canonical_from_coo(counts.size, k, rows, cols, rng.integers(-5, 6, rows.size), dup="first")
    blen = rng.choice([0, 1, 2, 40], k, p=[0.5, 0.3, 0.19, 0.01])
    B = canonical_from_coo(k, n, np.repeat(np.arange(k), blen), np.concatenate([rng.choice(n, c, replace=False) for c in blen]),
                           rng.integers(-5, 6, int(blen.sum())), dup="first")
    plan = spg.Plan()
    lo, hi = window or (None, None)
    a, b = to_dev(A, "i64"), to_dev(B, "i64")
    for _ in range(2):
        C = spg.spgemm(plan, "i64", a, b, lo, hi)
        check_full_vs_oracle(C, A, B, "i64", lo, hi)
    st = plan.stats()
    flops = oracle.row_flops(A, B, lo, hi)
    assert st["flops"] == flops.sum() and st["nnz_c"] == C.nnz
    assert sum(st["sym_rows"]) == sum(st["num_rows"]) == A.nrows
    assert sum(st["num_flops"]) == flops.sum() and sum(st["num_cnnz"]) == C.nnz
    inside = (A.col >= (lo or 0)) & (A.col < (k if hi is None else hi))
    assert sum(st["sym_annz"]) == sum(st["num_annz"]) == int(inside.sum())
    plan.close()


@pytest.mark.parametrize("spread", ["wide", "clustered", "doubled"])
@pytest.mark.parametrize("sr", ["f64", "i64", "bool"])
def test_sorted_product_rows(spread, sr):
    """Rows of the one-wave bins: product counts around the steps of 64 and
    the 128, 256 and 512 that a bin's rows may sort, more than 64 A entries,
    clustered columns (a bucket of more than 16) and runs of equal columns
    across steps; FP64 adds in ascending k and equals the oracle bit for bit."""
    rng = np.random.default_rng(5)
    K, n = 400, 30000
    blen = np.concatenate([rng.integers(0, 4, 300), rng.integers(4, 70, 100)])
    if spread == "wide":
        cols = [rng.choice(n, c, replace=False) for c in blen]
    elif spread == "clustered":
        cols = [np.concatenate([[0], 20000 + rng.choice(400, c - 1, replace=False)]) if c else [] for c in blen]
    else:
        cols = [7 * rng.choice(90, c, replace=False) for c in blen]
    br = np.repeat(np.arange(K), blen)
    B = canonical_from_coo(K, n, br, np.concatenate(cols).astype(np.int64), rng.uniform(-1, 1, br.size), dup="first")
    rows, acols = [], []
    targets = [65, 66, 127, 128, 129, 191, 192, 193, 255, 256, 257, 300, 383, 384, 385, 500, 511, 512, 513, 600]
    r = 0
    for t in targets * 3:
        ks, f = [], 0
        pool = rng.permutation(300 if r % 3 == 0 else K)  # every third row: short B rows, many A entries
        for k in pool:
            if blen[k] and f + blen[k] <= t:
                ks.append(k)
                f += blen[k]
        ks += [k for k in pool if blen[k] == 0][:5]
        rows += [r] * len(ks)
        acols += ks
        r += 1
    A = canonical_from_coo(r, K, np.array(rows), np.array(acols), rng.uniform(-1, 1, len(rows)), dup="first")
    if sr != "f64":
        kind = {"i64": "ones_i64", "bool": "true_bool"}[sr]
        A, B = synth.with_values(A, kind), synth.with_values(B, kind)
    # (no bitmap rows: n / 32 products and fewer)
    plan = spg.Plan()
    C = spg.spgemm(plan, sr, to_dev(A, sr), to_dev(B, sr))
    check_full_vs_oracle(C, A, B, sr)
    if sr == "f64":
        ref = oracle.spgemm(A, B, sr)
        flops = oracle.row_flops(A, B)
        cnt = np.diff(ref.row_ptr)
        # the rows a one-wave bin sorts: as many products as slots, three per two outputs
        slots = np.select([cnt <= 96, cnt <= 192, cnt <= 384], [128, 256, 512], 0)
        pick = np.repeat((flops <= slots) & (flops <= cnt + cnt // 2), cnt)
        assert pick.any() and np.array_equal(C.val.cpu().numpy()[pick], ref.val[pick])
    plan.close()


@pytest.mark.parametrize("layers", [2, 3, 4, 5, 8, 9, 16, 64])
@pytest.mark.parametrize("sr", ["f64", "i64", "bool"])
def test_merge_row_lengths(layers, sr):
    """Merge rows at the edges of their bins (64, 128, 384, 512 entries), empty
    layers first, last and in between, against the oracle bit for bit."""
    rng = np.random.default_rng(layers)
    sizes = [0, 1, 2, 63, 64, 65, 66, 127, 128, 129, 130, 255, 256, 257, 383, 384, 385, 511, 512, 513, 700]
    n = 5000
    parts = []
    owner = []
    for i, L in enumerate(sizes * 2):
        use = rng.choice(layers, max(1, layers // (1 + i % 3)), replace=False)  # some layers empty in the row
        owner.append(np.bincount(rng.choice(use, L), minlength=layers) if L else np.zeros(layers, int))
    for l in range(layers):
        lens = np.array([o[l] for o in owner])
        width = [n if i % 2 else 900 for i in range(len(lens))]  # narrow rows: many equal columns
        cols = [rng.choice(width[i], c, replace=False) for i, c in enumerate(lens)]
        rows = np.repeat(np.arange(len(lens)), lens)
        M = canonical_from_coo(len(lens), n, rows, np.concatenate(cols).astype(np.int64), rng.uniform(-1, 1, rows.size),
                               dup="first")
        parts.append(M if sr == "f64" else synth.with_values(M, {"i64": "ones_i64", "bool": "true_bool"}[sr]))
    plan = spg.Plan()
    ref = oracle.merge(parts, sr)
    for got in (spg.spgemm_merge_layers(plan, sr, [to_dev(M, sr) for M in parts]),
                spg.spgemm_merge_layers_noalloc(sr, [to_dev(M, sr) for M in parts])):
        rp, col, val = got.to_numpy()
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col) and np.array_equal(val, ref.val)
    plan.close()


@pytest.mark.parametrize("n", [60, 30000, (1 << 26) - 2, (1 << 26) + 5])
@pytest.mark.parametrize("sr", ["f64", "i64", "bool"])
def test_small_product_rows(n, sr):
    """Rows of up to 64 products: every count around the stages of the sort
    (2, 4 ... 64), B segments of 0, 1 and more, more than 64 A entries of empty B
    rows, runs of equal columns up to the whole row, odd numbers of rows, and
    columns on both sides of the 32-bit sort's limit.  FP64 adds in ascending k and
    equals the oracle bit for bit."""
    rng = np.random.default_rng(9)
    K = 700
    blen = np.concatenate([np.zeros(200, np.int64), np.ones(300, np.int64), rng.integers(2, 9, 150), rng.integers(9, 33, 50)])
    span = min(n, 60)
    cols = [np.concatenate([rng.choice(span, c - c // 2, replace=False), n - 1 - rng.choice(min(n // 2, 9000), c // 2, replace=False)])
            if n > 60 else rng.choice(n, c, replace=False) for c in blen]
    cols[200:260] = [np.array([n - 1])] * 60  # one column: runs as long as the row
    br = np.repeat(np.arange(K), blen)
    B = canonical_from_coo(K, n, br, np.concatenate(cols).astype(np.int64), rng.uniform(-1, 1, br.size), dup="first")
    rows, acols, r = [], [], 0
    for t in [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 60, 63, 64] * 3 + [64]:
        ks, f = [], 0
        pool = 200 + rng.permutation({0: 60, 1: 300, 2: 500}[r % 3])
        for k in pool:
            if f + blen[k] <= t:
                ks.append(k)
                f += blen[k]
        ks += list(rng.permutation(200)[:(0, 3, 120)[r // 2 % 3]])
        rows += [r] * len(ks)
        acols += ks
        r += 1
    A = canonical_from_coo(r, K, np.array(rows), np.array(acols), rng.uniform(-1, 1, len(rows)), dup="first")
    if sr != "f64":
        kind = {"i64": "ones_i64", "bool": "true_bool"}[sr]
        A, B = synth.with_values(A, kind), synth.with_values(B, kind)
    plan = spg.Plan()
    for lo, hi in [(None, None), (150, 420)]:
        C = spg.spgemm(plan, sr, to_dev(A, sr), to_dev(B, sr), lo, hi)
        check_full_vs_oracle(C, A, B, sr, lo, hi)
        assert oracle.row_flops(A, B, lo, hi).max() <= 64
        if sr == "f64":
            assert np.array_equal(C.val.cpu().numpy(), oracle.spgemm(A, B, sr, lo, hi).val)
    plan.close()


@pytest.mark.parametrize("sizes", [[2047, 1, 2048, 0, 2049, 3, 4095, 6144, 17], [5] * 1100])
@pytest.mark.parametrize("sr", ["f64", "i64", "bool"])
def test_batched_instance_edges(sizes, sr):
    """Batches whose instances begin and end at, before and after the copy's
    tiles of 2048 entries, and more instances than its tables hold; a second
    call with the values changed in place follows them."""
    rng = np.random.default_rng(4)
    dt = {"f64": np.float64, "i64": np.int64, "bool": np.uint8}[sr]
    draw = lambda k: (np.ones(k) if sr == "bool" else rng.integers(1, 5, k)).astype(dt)
    inst = []
    for nnz in sizes:
        n, m = max(5, nnz // 7), max(2, nnz // 40)
        flat = rng.choice(n * n, nnz, replace=False)
        A = canonical_from_coo(n, n, flat // n, flat % n, draw(nnz), dup="first")
        agg = rng.integers(0, m, n)
        R = canonical_from_coo(n, m, np.arange(n), agg, draw(n), dup="first")
        RT = canonical_from_coo(m, n, agg, np.arange(n), draw(n), dup="first")
        inst.append([RT, A, R])
    plan = spg.Plan()
    dev = [[to_dev(M, sr) for M in t] for t in inst]
    for again in range(3):
        if again:
            for t, d in zip(inst, dev):
                t[1].val[:] = draw(t[1].nnz)
                d[1].val.copy_(torch.from_numpy(t[1].val))
        got = spg.spgemm_galerkin_batched(plan, sr, *[[d[k] for d in dev] for k in range(3)]).fetch(plan)
        for b, (C, (RT, A, R)) in enumerate(zip(got, inst)):
            ref = oracle.spgemm(oracle.spgemm(RT, A, sr), R, sr)
            assert np.array_equal(C.row_ptr.cpu().numpy(), ref.row_ptr) and np.array_equal(C.col.cpu().numpy(), ref.col), b
            assert np.array_equal(C.val.cpu().numpy(), ref.val), b  # small integers: exact
    plan.close()
