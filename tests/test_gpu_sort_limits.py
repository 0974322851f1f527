"""Sorted rows at the limit of their packing: a column's distance from the row's
first one and the entry's place share 32 bits, which columns 0 and 2^23 - 1 fill
(entry 511 of the last column is the all-ones word that pads the sort).  One
column more takes the other kernels.  Bit for bit against the oracle."""

import numpy as np
import pytest

import oracle
import paper_1510_00844_amd as spg
import synth
from gpu_util import check_full_vs_oracle, to_dev
from synth.gen import canonical_from_coo

pytestmark = pytest.mark.gpu

LIMIT = 1 << 23
SIZES = [65, 128, 129, 255, 256, 257, 384, 511, 512]


def entries(n, size, distinct, spread, rng):
    """`size` columns of `distinct` different ones, 0 first and n - 1 last."""
    if spread == "wide":
        pool = 1 + rng.choice(n - 2, distinct - 2, replace=False)
    else:  # most in one cluster, near the start, the middle or the end
        pool = int(rng.choice([1, n // 2, n - 700])) + rng.choice(690, distinct - 2, replace=False)
    extra = rng.choice(pool, size - distinct) if size > distinct else np.zeros(0, np.int64)
    mid = np.concatenate([pool, extra])
    rng.shuffle(mid)
    return np.concatenate([[0], mid, [n - 1]])


def split(cols, parts, rng):
    """The entries in order over `parts` sorted, duplicate-free sets (the last
    one holds the last entry)."""
    out = [[] for _ in range(parts)]
    for j in cols[1:-1]:
        for p in rng.permutation(parts):
            if j not in out[p]:
                out[p].append(int(j))
                break
        else:
            raise AssertionError("a column too often")
    out[0].append(int(cols[0]))
    out[-1].append(int(cols[-1]))
    return [np.unique(x).astype(np.int64) for x in out]


@pytest.mark.parametrize("n", [LIMIT, LIMIT + 1])
@pytest.mark.parametrize("spread", ["wide", "clustered"])
@pytest.mark.parametrize("sr", ["f64", "i64", "bool"])
def test_product_rows_at_the_packing_limit(n, spread, sr):
    print("case packing limit, product", n, spread, sr, flush=True)
    rng = np.random.default_rng(12)
    b_rows, a_rows = [], []
    for size in SIZES:
        for distinct in (min(size, 380), min(size - 1, (2 * size + 5) // 3)):
            parts = split(entries(n, size, distinct, spread, rng), 7, rng)
            a_rows.append(range(len(b_rows), len(b_rows) + 7))
            b_rows += parts
    K = len(b_rows)
    rows = np.repeat(np.arange(K), [len(b) for b in b_rows])
    B = canonical_from_coo(K, n, rows, np.concatenate(b_rows), rng.uniform(-1, 1, rows.size), dup="first")
    ar = np.repeat(np.arange(len(a_rows)), 7)
    A = canonical_from_coo(len(a_rows), K, ar, np.concatenate([list(r) for r in a_rows]), rng.uniform(-1, 1, ar.size), dup="first")
    flops, cnt = oracle.row_flops(A, B), np.diff(oracle.spgemm(A, B, "bool", values=False).row_ptr)
    assert flops.max() == 512 and flops.min() == 65 and (2 * flops <= 3 * cnt).all()
    if sr != "f64":
        kind = {"i64": "ones_i64", "bool": "true_bool"}[sr]
        A, B = synth.with_values(A, kind), synth.with_values(B, kind)
    plan = spg.Plan()
    C = spg.spgemm(plan, sr, to_dev(A, sr), to_dev(B, sr))
    check_full_vs_oracle(C, A, B, sr)
    if sr == "f64" and n == LIMIT:  # sorted rows add in ascending k
        ref = oracle.spgemm(A, B, sr)
        table = np.select([cnt <= 96, cnt <= 192, cnt <= 384], [128, 256, 512], 0)
        pick = np.repeat((flops > 64) & (flops <= table), cnt)
        assert pick.mean() > 0.5 and np.array_equal(C.val.cpu().numpy()[pick], ref.val[pick])
    plan.close()


@pytest.mark.parametrize("n", [LIMIT, LIMIT + 1])
@pytest.mark.parametrize("spread", ["wide", "clustered"])
@pytest.mark.parametrize("c", [9, 16])
def test_merge_rows_at_the_packing_limit(n, spread, c):
    print("case packing limit, merge", n, spread, c, flush=True)
    rng = np.random.default_rng(13)
    per = [([], []) for _ in range(c)]
    r = 0
    for size in SIZES:
        for distinct in (size, size // 2 + 1):
            for l, cols in enumerate(split(entries(n, size, distinct, spread, rng), c, rng)):
                per[l][0].append(np.full(len(cols), r))
                per[l][1].append(cols)
            r += 1
    hl = []
    for rows, cols in per:
        rows, cols = np.concatenate(rows), np.concatenate(cols)
        hl.append(canonical_from_coo(r, n, rows, cols, rng.uniform(-1, 1, rows.size), dup="first"))
    assert sum(np.diff(M.row_ptr) for M in hl).max() == 512
    ref = oracle.merge(hl, "f64")
    plan = spg.Plan(profile=True)
    dev = [to_dev(M) for M in hl]
    for got in (spg.spgemm_merge_layers(plan, "f64", dev), spg.spgemm_merge_layers_noalloc("f64", dev)):
        rp, col, val = got.to_numpy()
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col) and np.array_equal(val, ref.val)
    assert ("merge_sort" in plan.profile_read()) == (n == LIMIT)
    plan.close()
