"""The rank-chunk items' size, as the host computes it for the launch, over every
legal column chunk and chunk group: within the dynamic LDS that the kernel is
declared with, at least one chunk of outputs, fewer outputs than the 16-bit
ranks count."""

import os
import subprocess

import pytest

from paper_1510_00844_amd import build as hip_build

SOURCE = r"""
#include "numeric.hpp"
#include <cstdio>
using namespace spg;
int main() {
    long bad = 0, cases = 0, largest = 0;
    for (int64_t max_lds : {163840, 65536})
        for (int32_t W : {2048, 4096, 8192, 16384})
            for (int32_t group = 1; group <= 256; ++group)
                for (int64_t n : {2049, 4097, 20011, 65536, 100000, 200003, 262144, 400000, 524288}) {
                    if (W * 8 + RANKC_STATIC_LDS + W / 32 * 6 > max_lds) continue;
                    const int32_t chunks = (int32_t)((n + W - 1) / W);
                    for (int64_t nr : {1, 64, 5000})
                        for (int64_t per = 1; per <= n; per = per * 9 / 8 + 1) {
                            const RankShape s = rankc_shape(nr, nr * per, chunks, group, W, max_lds);
                            const int64_t lds = (int64_t)s.RC * 8 + (int64_t)s.G * (W / 32) * 6;
                            ++cases;
                            if (lds > largest) largest = lds;
                            if (lds > rankc_dyn_lds(max_lds) || s.RC < W || s.RC >= 65536 || s.G < 1 ||
                                s.G > group || s.G > chunks)
                                if (++bad <= 5)
                                    std::printf("max_lds %ld W %d group %d n %ld rows %ld outputs %ld: RC %d G %d lds %ld of %ld\n",
                                                (long)max_lds, W, group, (long)n, (long)nr, (long)per, s.RC, s.G, (long)lds,
                                                (long)rankc_dyn_lds(max_lds));
                        }
                }
    std::printf("cases %ld bad %ld largest %ld\n", cases, bad, largest);
    return bad != 0;
}
"""


def test_rank_chunk_items_fit_their_declared_lds(tmp_path):
    try:
        cc = hip_build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "shapes.hip", tmp_path / "shapes"
    src.write_text(SOURCE)
    flags = [f for f in hip_build.flags() if f not in ("-fPIC", "-shared")]
    r = subprocess.run([cc] + flags + ["-I" + hip_build.CSRC, "-o", str(exe), str(src)],
                       capture_output=True, text=True, cwd=os.path.dirname(hip_build.CSRC))
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
