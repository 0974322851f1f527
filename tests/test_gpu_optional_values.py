"""Matrices without a value array: boolean matrices, where it means that every
stored entry is true, beside others that hold truth values; and any matrix
where only the structure of the result is asked for."""

import numpy as np
import pytest

import oracle
import paper_1510_00844_amd as spg
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
