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
