"""Product rows of the one-wave bins whose columns lie in clusters (B rows that
are runs of neighbouring columns): the buckets of equal width overflow, and the
ranks of a bitmap take over where the span allows it, else a sort of the whole
row.  FP64 adds in ascending k and equals the oracle bit for bit; clustered rows
take at most a few times as long as spread ones."""

import numpy as np
import pytest
import torch

import oracle
import paper_1510_00844_amd as spg
import synth
from gpu_util import check_full_vs_oracle, to_dev
from synth.gen import canonical_from_coo

pytestmark = pytest.mark.gpu

N = 60000


def clustered(slots, seed):
    """Rows of the bin of `slots`: clusters of runs from a base column on, the last
    column at, just inside and just past what a bitmap of `slots` words spans; the
    runs' lengths, their overlaps (equal columns) and the row's size vary."""
    rng = np.random.default_rng(seed)
    limit = 3 * slots // 4  # outputs of the bin's rows
    b_rows, a_rows, r = [], [], 0
    for span in (32 * slots - 1, 32 * slots, 32 * slots + 1, 6000 * slots // 512, 40 * slots, 2 * slots):
        for run in (17, 24, 33, 60):
            for clusters in (2, 3, 8, 64):
                for total in (limit // 2 + 3, limit - 5):
                    base = int(rng.integers(0, N - 64 * slots - 1))
                    count = max(2, total // run)
                    at = np.sort(rng.integers(0, span - run + 1, clusters))
                    ks = []
                    for t in range(count):
                        s = 0 if t == 0 else (span - run if t == 1 else min(span - run, int(at[t % clusters]) + (t // clusters) * (run - t % 3)))
                        ks.append(len(b_rows))
                        b_rows.append(base + s + np.arange(run))
                    if total == limit - 5:  # a few equal columns, added in the order of k
                        ks.append(len(b_rows))
                        b_rows.append(np.sort(rng.choice(b_rows[ks[-2]], 9, replace=False)))
                    a_rows.append(ks)
                    r += 1
    K = len(b_rows)
    rows = np.repeat(np.arange(K), [len(b) for b in b_rows])
    perm = rng.permutation(K)
    inv = np.argsort(perm)
    B = canonical_from_coo(K, N, perm[rows], np.concatenate(b_rows), rng.uniform(-1, 1, rows.size), dup="first")
    ar = np.repeat(np.arange(r), [len(k) for k in a_rows])
    ac = perm[np.concatenate([np.array(k) for k in a_rows])]
    assert inv[perm].tolist() == list(range(K))
    return canonical_from_coo(r, K, ar, ac, rng.uniform(-1, 1, ar.size), dup="first"), B


@pytest.mark.parametrize("slots", [128, 256, 512])
@pytest.mark.parametrize("sr", ["f64", "i64", "bool"])
def test_clustered_rows(slots, sr):
    print("case clustered rows", slots, sr, flush=True)
    A, B = clustered(slots, slots)
    if sr != "f64":
        kind = {"i64": "ones_i64", "bool": "true_bool"}[sr]
        A, B = synth.with_values(A, kind), synth.with_values(B, kind)
    plan = spg.Plan()
    C = spg.spgemm(plan, sr, to_dev(A, sr), to_dev(B, sr))
    check_full_vs_oracle(C, A, B, sr)
    assert plan.stats()["num_rows"][3 + {128: 0, 256: 1, 512: 2}[slots]] > A.nrows // 3
    if sr == "f64":
        ref = oracle.spgemm(A, B, sr)
        cnt = np.diff(ref.row_ptr)
        flops = oracle.row_flops(A, B)
        table = np.select([cnt <= 96, cnt <= 192, cnt <= 384], [128, 256, 512], 0)
        pick = np.repeat((flops > 64) & (flops <= table) & (flops <= cnt + cnt // 2), cnt)
        assert pick.mean() > 0.5 and np.array_equal(C.val.cpu().numpy()[pick], ref.val[pick])
    plan.close()


def test_clustered_rows_take_no_longer_than_hashed_ones():
    """12 runs of 32 columns in a window of 12000 (384 outputs a row) against 24
    rows of 16 columns spread over all of them: the kernel's times."""
    m = 1 << 16
    rng = np.random.default_rng(3)
    ids = np.arange(m)

    def of_rows(cols):
        return canonical_from_coo(m, m, np.repeat(ids, cols.shape[1]), cols.ravel(), rng.random(cols.size), dup="first")

    runs = of_rows(np.minimum(ids, m - 32)[:, None] + np.arange(32))
    near = of_rows(np.minimum(np.maximum(ids - 6000, 0)[:, None] + np.arange(12) * 1000 + rng.integers(0, 968, (m, 12)), m - 1))
    spread = of_rows(rng.integers(0, m, (m, 16)))
    far = of_rows(rng.integers(0, m, (m, 24)))
    times = []
    for A, B in ((far, spread), (near, runs)):
        plan = spg.Plan(profile=True, streams=1)
        a, b = to_dev(A), to_dev(B)
        best = float("inf")
        for _ in range(6):
            plan.profile_reset()
            spg.spgemm(plan, "f64", a, b)
            torch.cuda.synchronize()
            best = min(best, sum(t for k, (_, t) in plan.profile_read().items() if k.startswith("num_hash")))
        times.append(best)
        plan.close()
    print("num_hash: spread %.3f ms, clustered %.3f ms" % tuple(times))
    assert times[1] < 2 * times[0]
