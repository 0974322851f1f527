"""Long rows that lie side by side are spread over the GPU: a kernel over 64 of
them takes a few times as long as over one, not 64 times.  Launch times come from
the plan's profile; the best of several calls is compared."""

import numpy as np
import pytest
import torch

import oracle
import paper_1510_00844_amd as spg
from gpu_util import check_full_vs_oracle, to_dev
from synth.gen import canonical_from_coo

pytestmark = pytest.mark.gpu

SPREAD = 8.0  # 64 rows one after another would be 64


def kernel_ms(plan, name, call, reps=7):
    """Shortest time of the kernel's launches in one call."""
    call()
    best = float("inf")
    for _ in range(reps):
        plan.profile_reset()
        call()
        torch.cuda.synchronize()
        best = min(best, plan.profile_read()[name][1])
    return best


def restrict(plan, sizes, seed=3):
    agg = np.random.default_rng(seed).permutation(np.repeat(np.arange(len(sizes)), sizes)).astype(np.int32)
    dev = torch.from_numpy(agg).cuda()
    return agg, lambda: spg.spg_restriction(plan, "f64", dev, len(sizes))


def test_long_restriction_rows_side_by_side():
    plan = spg.Plan(profile=True)
    one = kernel_ms(plan, "sort_row_cols", restrict(plan, [4096])[1])
    many = kernel_ms(plan, "sort_row_cols", restrict(plan, [4096] * 64)[1])
    print("sort_row_cols: 1 row %.3f ms, 64 rows %.3f ms" % (one, many))
    assert many < SPREAD * one
    plan.close()


@pytest.mark.parametrize("sizes", [
    [64, 65, 127, 128, 129, 255, 256, 257, 1, 511, 512, 513, 2047, 2049, 4095, 4096],
    [1] * 3000 + [300, 4000, 257, 70] * 40 + [2] * 3000,
    [1] * 70000 + [257, 600, 65] * 6 + [1] * 70000 + [1025, 256, 300],
])
def test_restriction_rows_of_every_sort(sizes):
    """R^T rows of the register, the wave and the workgroup sort, more rows than
    the long rows' kernel has workgroups, and than it looks at in one step."""
    plan = spg.Plan()
    agg, call = restrict(plan, sizes)
    R, RT = call()
    assert np.array_equal(RT.row_ptr.cpu().numpy(), np.concatenate([[0], np.cumsum(sizes)]))
    assert np.array_equal(RT.col.cpu().numpy(), np.argsort(agg, kind="stable"))
    assert np.array_equal(R.col.cpu().numpy(), agg)
    plan.close()


def rows_of_lengths(lens, K, seed):
    """A matrix of K columns whose row i holds lens[i] entries."""
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens)
    cols = [rng.permutation(K)[:c] if c > 64 else rng.choice(K, c, replace=False) for c in lens[lens > 8]]
    out = np.empty(lens.sum(), np.int64)
    big = np.repeat(lens > 8, lens)
    if cols:
        out[big] = np.concatenate(cols)
    out[~big] = (np.repeat(rng.integers(0, K, lens.size), lens) + 911 * (np.arange(lens.sum()) - np.repeat(np.cumsum(lens) - lens, lens)))[~big] % K
    rows = np.repeat(np.arange(lens.size), lens)
    return canonical_from_coo(lens.size, K, rows, out, rng.integers(1, 5, rows.size), dup="first")


@pytest.mark.parametrize("name,one,many", [
    ("hub rows among short ones", [30000] + [4] * 20000, [30000] * 64 + [4] * 20000),
    ("few rows, all long", [3000] * 4, [3000] * 1000),
])
def test_row_analysis_of_long_rows_side_by_side(name, one, many):
    K = 40009
    B = to_dev(rows_of_lengths([2] * K, 5000, 1), "i64")
    plan = spg.Plan(profile=True)
    times = []
    for lens in (one, many):
        A = to_dev(rows_of_lengths(lens, K, 2), "i64")
        times.append(kernel_ms(plan, "rowinfo", lambda: spg.spgemm_symbolic(plan, "i64", A, B)))
    print("rowinfo, %s: %.4f ms, %.4f ms" % (name, *times))
    assert times[1] < SPREAD * times[0]
    plan.close()


@pytest.mark.parametrize("m", [3, 1000, 262144, 262145, 300001])
def test_row_analysis_deals_out_every_row(m):
    """Rows of every length class at the first rows, the last and around the
    runs, in numbers of rows on both sides of the longer runs; the bin counts see
    every row once."""
    K, n = 6000, 900
    lens = np.ones(m, np.int64)
    special = [5000, 2049, 2048, 129, 128, 0, 17, 300]
    for base in (0, 12, 62, m // 2, m - 9):
        for k, c in enumerate(special):
            if 0 <= base + k < m:
                lens[base + k] = c
    A = rows_of_lengths(lens, K, 5)
    B = rows_of_lengths([1, 0, 3] * (K // 3), n, 6)
    plan = spg.Plan()
    a, b = to_dev(A, "i64"), to_dev(B, "i64")
    for lo, hi in ((0, K), (900, 5100)):
        check_full_vs_oracle(spg.spgemm(plan, "i64", a, b, lo, hi), A, B, "i64", lo, hi)
        st = plan.stats()
        assert sum(st["sym_rows"]) == m and st["flops"] == oracle.row_flops(A, B, lo, hi).sum()
    plan.close()
