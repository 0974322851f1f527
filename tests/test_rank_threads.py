"""Threads of the whole-row rank kernel: an explicit option is kept, the default
follows the row's LDS."""

import os
import subprocess

import pytest

from paper_1510_00844_amd import build as hip_build

SOURCE = r"""
#include "numeric.hpp"
#include <cstdio>
using namespace spg;
int main() {
    const int64_t max_lds = 163840;
    int bad = 0;
    for (int64_t cap : {4096, 8192, 16384})
        for (int64_t value : {4, 8})
            for (int64_t n = 64; n <= (1 << 19); n = n * 5 / 4) {
                const int64_t lds = (n + 31) / 32 * 6 + cap * value;
                if (lds + RANK_STATIC_LDS > max_lds) continue;
                const bool fits = lds + RANK_STATIC_LDS_1024 <= max_lds, one = 2 * (lds + RANK_STATIC_LDS) > max_lds;
                bad += rank_threads(512, lds, max_lds) != 512;
                bad += rank_threads(1024, lds, max_lds) != (fits ? 1024 : 512);
                bad += rank_threads(0, lds, max_lds) != (one && fits ? 1024 : 512);
            }
    std::printf("%d wrong\n", bad);
    return bad != 0;
}
"""


def test_rank_threads(tmp_path):
    try:
        cc = hip_build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "threads.hip", tmp_path / "threads"
    src.write_text(SOURCE)
    flags = [f for f in hip_build.flags() if f not in ("-fPIC", "-shared")]
    r = subprocess.run([cc] + flags + ["-I" + hip_build.CSRC, "-o", str(exe), str(src)], capture_output=True, text=True,
                       cwd=os.path.dirname(hip_build.CSRC))
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
