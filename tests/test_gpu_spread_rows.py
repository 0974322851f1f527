"""Long rows that lie side by side are spread over the GPU: a kernel over 64 of
them takes a few times as long as over one, not 64 times.  Launch times come from
the plan's profile; the best of several calls is compared."""

import numpy as np
import pytest
import torch

import paper_1510_00844_amd as spg

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
