"""Rank-chunk items at the ends of their range: the largest that the LDS takes
(one workgroup per CU), and items of more bitmap words than the workgroup holds in
registers, whose ranks are laid out tile by tile."""

import numpy as np
import pytest

import oracle
import paper_1510_00844_amd as spg
from gpu_util import check_full_vs_oracle, to_dev
from synth.gen import canonical_from_coo

pytestmark = pytest.mark.gpu

THREADS = 512          # of the rank-chunk kernel
WORDS = 8 * THREADS    # bitmap words it holds in registers
STATIC_LDS = 9176      # its static LDS, as the host reckons it
MAX_LDS = 163840


def item_shape(rows, outputs, chunks, group, W):
    """(outputs, chunks) of an item, by the rule of the library."""
    def g_of(RC):
        g = min((2 * RC * rows * chunks + outputs) // (2 * outputs), chunks, group)
        return max(g, 1)

    def lds(RC, G):
        return RC * 8 + G * (W // 32) * 6 + STATIC_LDS

    RC = max(W, 4096)
    G = g_of(RC)
    while G > 1 and lds(RC, G) > MAX_LDS:
        G -= 1
    wg = min(max(MAX_LDS // lds(RC, G), 1), 4)
    while G < chunks and G < group and RC + 512 < 65536 and lds(RC + 512, g_of(RC + 512)) * wg <= MAX_LDS:
        RC += 512
        G = g_of(RC)
    return RC, G


def heavy_rows(n, distinct, per_row, blen, seed):
    """A of a few heavy rows and B of even rows whose columns are `distinct` of the
    n, spread over all of them."""
    rng = np.random.default_rng(seed)
    K = 3000
    pool = np.sort(rng.choice(n, distinct, replace=False))
    rows = np.repeat(np.arange(len(per_row)), per_row)
    cols = np.concatenate([rng.choice(K, c, replace=False) for c in per_row])
    A = canonical_from_coo(len(per_row), K, rows, cols, rng.uniform(-1, 1, rows.size), dup="first")
    br = np.repeat(np.arange(K), blen)
    bc = pool[rng.integers(0, distinct, br.size)]
    return A, canonical_from_coo(K, n, br, bc, rng.uniform(-1, 1, br.size), dup="first")


CASES = {
    # more than 4096 words an item: several tiles
    "tiles": (dict(dense_chunk_cols=2048, chunk_group=256, rank_max_nnz=1, chunk_min_nnz=1), 200003, 3000,
              [500, 700, 900, 449, 1345, 2900], 16),
    # the item takes all the LDS that the kernel is declared with
    "largest": (dict(dense_chunk_cols=8192), 100000, 23500, [2700, 2800, 2900, 3000, 2750, 2850], 28),
}


@pytest.mark.parametrize("case", list(CASES))
def test_rank_chunk_item_shapes(case):
    print("case rank-chunk shapes", case, flush=True)
    opts, n, distinct, per_row, blen = CASES[case]
    A, B = heavy_rows(n, distinct, per_row, blen, seed=8)
    plan = spg.Plan(**opts)
    for sr in ("f64", "i64"):
        if sr == "i64":
            A.val, B.val = np.rint(A.val * 9).astype(np.int64), np.rint(B.val * 9).astype(np.int64)
        a, b = to_dev(A, sr), to_dev(B, sr)
        for _ in range(2):
            check_full_vs_oracle(spg.spgemm(plan, sr, a, b), A, B, sr)
        st = plan.stats()
        rows, outputs = st["num_rows"][11], st["num_cnnz"][11]
        assert rows == A.nrows
        W = opts["dense_chunk_cols"]
        RC, G = item_shape(rows, outputs, -(-n // W), opts.get("chunk_group", 32), W)
        if case == "tiles":
            assert G * (W // 32) > WORDS
        else:
            assert RC * 8 + G * (W // 32) * 6 > MAX_LDS - STATIC_LDS - 4096
    plan.close()
