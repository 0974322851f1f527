"""Which kernels a merge of five to eight layers takes, by its rows and their mean
length, and that its result is the oracle's bit for bit on either side of each line."""

import numpy as np
import pytest
import torch

import oracle
import paper_1510_00844_amd as spg
import synth
from gpu_util import to_dev
from synth import CSR
from synth.gen import canonical_from_coo

pytestmark = pytest.mark.gpu


def make_layers(c, m, mean, seed):
    """c layers over m rows of about `mean` entries altogether, at most `mean` on
    average; some rows empty, short, and above 512 entries; equal columns."""
    rng = np.random.default_rng(seed)
    n = 4000
    lens = rng.integers(0, max(2, 2 * mean // c - 1), (c, m))
    lens[:, rng.choice(m, 7, replace=False)] = 0
    lens[:, rng.choice(m, 5, replace=False)] = 1
    lens[:, rng.choice(m, 3, replace=False)] = 110
    lens[:, rng.choice(m, 9, replace=False)] = 30
    out = []
    for l in range(c):
        rows = np.repeat(np.arange(m), lens[l])
        cols = rng.integers(0, n, rows.size)
        out.append(canonical_from_coo(m, n, rows, cols, rng.uniform(-1, 1, rows.size), dup="first"))
    return out


# (rows, mean entries a row, whether rows are sorted)
LINES = [(2048, 16, False), (8191, 16, False), (8192, 16, True), (8192, 100, False), (16383, 80, False),
         (16384, 80, True), (16384, 410, False)]


@pytest.mark.parametrize("m,mean,sorts", LINES)
@pytest.mark.parametrize("c", [5, 8])
def test_merge_route(c, m, mean, sorts):
    print("case merge route", c, m, mean, flush=True)
    hl = make_layers(c, m, mean, seed=c + m)
    if mean > 384:
        assert sum(M.nnz for M in hl) > 384 * m
    plan = spg.Plan(profile=True)
    dev = [to_dev(M) for M in hl]
    got = spg.spgemm_merge_layers(plan, "f64", dev)
    torch.cuda.synchronize()
    names = set(plan.profile_read())
    assert ({"merge_sort", "merge_small"} <= names) == sorts and ("merge_kway" in names) != sorts
    ref = oracle.merge(hl, "f64")
    for g in (got, spg.spgemm_merge_layers_noalloc("f64", dev)):
        rp, col, val = g.to_numpy()
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col) and np.array_equal(val, ref.val)
    plan.close()


@pytest.mark.parametrize("c", [5, 8])
def test_sorted_merge_of_optional_values(c):
    """The sorted rows of five to eight layers: boolean layers with and without
    truth values, and structure alone."""
    print("case sorted merge, optional values", c, flush=True)
    hl = make_layers(c, 16384, 80, seed=90 + c)
    rng = np.random.default_rng(c)
    for M in hl:
        M.val = (rng.random(M.nnz) < 0.3).astype(np.uint8)
    bare = [CSR(M.nrows, M.ncols, M.row_ptr, M.col, None if l % 2 else M.val) for l, M in enumerate(hl)]
    ref = oracle.merge([synth.with_values(M, "true_bool") if l % 2 else M for l, M in enumerate(hl)], "bool")
    plan = spg.Plan(profile=True)
    dev = [to_dev(M, "bool") for M in bare]
    for got in (spg.spgemm_merge_layers(plan, "bool", dev), spg.spgemm_merge_layers_noalloc("bool", dev)):
        rp, col, val = got.to_numpy()
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(col, ref.col) and np.array_equal(val, ref.val)
    assert "merge_sort" in plan.profile_read()
    none = [to_dev(CSR(M.nrows, M.ncols, M.row_ptr, M.col, None)) for M in hl]
    got = spg.spgemm_merge_layers(plan, "i64", none, values=False)
    assert torch.equal(got.row_ptr.cpu(), torch.from_numpy(ref.row_ptr)) and torch.equal(got.col.cpu(), torch.from_numpy(ref.col))
    plan.close()
