"""Matrices without a value array: boolean matrices, where it means that every
stored entry is true, beside others that hold truth values; and any matrix
where only the structure of the result is asked for."""

import numpy as np
import pytest

import oracle
import paper_1510_00844_amd as spg
import synth
from gpu_util import to_dev
from synth import CSR
from synth.gen import canonical_from_coo

pytestmark = pytest.mark.gpu

# merge rows on both sides of the bins' limits: the wave kernels to 64, 384 and
# 512 entries, the rank kernels to 4096, the column chunks above
MERGE_ROWS = [0, 1, 2, 33, 63, 64, 65, 66, 127, 129, 200, 383, 385, 400, 511, 512, 513, 900, 1500, 4300]


def merge_layers_of(c, seed):
    """c boolean layers whose row i holds MERGE_ROWS[i] entries over all of
    them, with truth values of both kinds; every third row leaves layers empty."""
    rng = np.random.default_rng(seed)
    n, sizes = 6000, MERGE_ROWS * 2
    owner = []
    for i, L in enumerate(sizes):
        use = rng.choice(c, max(2, c // 2) if i % 3 == 0 and L < 1000 else c, replace=False)
        owner.append(np.bincount(rng.choice(use, L), minlength=c))
    out = []
    for l in range(c):
        lens = np.array([o[l] for o in owner])
        cols = [rng.choice(n if i % 2 or k > 800 else 900, k, replace=False) for i, k in enumerate(lens)]
        rows = np.repeat(np.arange(len(sizes)), lens)
        vals = (rng.random(rows.size) < 0.3).astype(np.uint8)
        out.append(canonical_from_coo(len(sizes), n, rows, np.concatenate(cols).astype(np.int64), vals, dup="first"))
    return out


def without_values(M):
    return CSR(M.nrows, M.ncols, M.row_ptr, M.col, None)


@pytest.mark.parametrize("c", [2, 4, 5, 8, 9, 16, 64])
@pytest.mark.parametrize("bare", ["even", "odd", "last", "first"])
def test_merge_of_boolean_layers_with_and_without_values(c, bare):
    """Some layers hold truth values (false among them) and others none: an
    entry of a layer without values is true, wherever its neighbours in the
    row come from."""
    print("case mixed boolean merge", c, bare, flush=True)
    full = merge_layers_of(c, 40 + c)
    none = {"even": range(0, c, 2), "odd": range(1, c, 2), "last": [c - 1], "first": [0]}[bare]
    hl = [without_values(M) if l in none else M for l, M in enumerate(full)]
    ones = [CSR(M.nrows, M.ncols, M.row_ptr, M.col, np.ones(M.nnz, np.uint8)) if l in none else M
            for l, M in enumerate(full)]
    ref = oracle.merge(ones, "bool")
    assert 0 < int(ref.val.sum()) < ref.nnz  # both truth values in the result
    plan = spg.Plan()
    dev = [to_dev(M, "bool") for M in hl]
    for got in (spg.spgemm_merge_layers(plan, "bool", dev), spg.spgemm_merge_layers_noalloc("bool", dev)):
        rp, col, val = got.to_numpy()
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col)
        assert np.array_equal(val, ref.val)
    plan.close()


@pytest.mark.parametrize("c", [2, 5, 8, 9, 16])
@pytest.mark.parametrize("sr", ["f64", "i64", "bool"])
def test_merge_of_structure_alone(c, sr):
    """Layers without values, merged without values, in every bin."""
    print("case structure-only merge", c, sr, flush=True)
    hl = [without_values(M) for M in merge_layers_of(c, 60 + c)]
    ref = oracle.merge(hl, "bool")
    plan = spg.Plan()
    dev = [to_dev(M) for M in hl]
    for got in (spg.spgemm_merge_layers(plan, sr, dev, values=False),
                spg.spgemm_merge_layers_noalloc(sr, dev, values=False)):
        rp, col, val = got.to_numpy()
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col) and val is None
    plan.close()


PRODUCT_OPTS = {
    "default": {},
    "rank_chunks": dict(rank_max_nnz=1, chunk_min_nnz=1, dense_chunk_cols=2048),
    "dense": dict(hash_max_nnz=64),
    "heap": dict(heap_max_lists=32),
}


@pytest.mark.parametrize("opts", list(PRODUCT_OPTS))
@pytest.mark.parametrize("sr", ["f64", "i64", "bool"])
def test_product_structure_alone(opts, sr):
    """Operands without values, multiplied without values: rows of one A entry
    and more, of every accumulator, on both sides of the one-bitmap width, full and
    windowed."""
    print("case structure-only product", opts, sr, flush=True)
    rng = np.random.default_rng(7)
    A = synth.rmat(11, 8, synth.G500, seed=21)
    wide = 700001
    rows = np.repeat(np.arange(A.ncols), 6)
    near = rng.integers(0, 40, (A.ncols, 1)) * 17000 + rng.integers(0, 900, (A.ncols, 6))
    W = canonical_from_coo(A.ncols, wide, rows, near.ravel(), np.ones(rows.size), dup="first")
    plan = spg.Plan(**PRODUCT_OPTS[opts])
    bins = np.zeros(17, np.int64)
    for B in (synth.rmat(11, 8, synth.SSCA, seed=22), W):
        a, b = to_dev(without_values(A)), to_dev(without_values(B))
        for lo, hi in ((0, A.ncols), (100, 1400)):
            C = spg.spgemm(plan, sr, a, b, lo, hi, values=False)
            bins += np.array(plan.stats()["num_rows"])
            ref = oracle.spgemm(A, B, "bool", lo, hi, values=False)
            assert C.val is None
            assert np.array_equal(C.row_ptr.cpu().numpy(), ref.row_ptr) and np.array_equal(C.col.cpu().numpy(), ref.col)
    assert bins[1] > 0 and bins[2] > 0  # the tiny and the small rows
    assert {"default": bins[3:12].sum(), "rank_chunks": bins[11], "dense": bins[12], "heap": bins[16]}[opts] > 0
    plan.close()
