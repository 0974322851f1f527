"""The rules that spread a pass's kernels over the helper streams, on their lines."""

import os
import subprocess

import pytest

from paper_1510_00844_amd import build as hip_build

SOURCE = r"""
#include "rowinfo.hpp"
#include <cstdio>
#include <initializer_list>
using namespace spg;
static int failed = 0;
static void expect(const char* what, std::initializer_list<int> bins, int64_t products, int first_bin, bool want) {
    int64_t c[2 * NBINS] = {};
    for (int b : bins) {
        c[b] = 10;
        c[NBINS + b] = products / (int64_t)bins.size() + 1;
    }
    if (worth_forking(c, first_bin) != want) {
        std::printf("%s: not %d\n", what, (int)want);
        ++failed;
    }
}
// numeric bins with the given shares of 2^22 products
static void numeric(const char* what, std::initializer_list<int> bins, std::initializer_list<double> shares, bool sym,
                    bool want) {
    int64_t c[2 * NBINS] = {};
    auto s = shares.begin();
    for (int b : bins) {
        c[b] = 1;
        c[NBINS + b] = (int64_t)(*s++ * (1 << 22));
    }
    if (worth_forking_numeric(c, sym) != want) {
        std::printf("numeric, %s: not %d\n", what, (int)want);
        ++failed;
    }
}
int main() {
    const int64_t many = 1 << 20, few = many - 100;
    expect("five kernels", {2, 3, 4, 5, 12}, many, BIN_SMALL, false);
    expect("five, and rows of one A entry", {1, 2, 3, 4, 5, 12}, many, BIN_SMALL, false);
    expect("five, and rows of one A entry with a kernel", {1, 2, 3, 4, 5, 12}, many, BIN_TINY, true);
    expect("five, and empty rows", {0, 2, 3, 4, 5, 12}, many, BIN_TINY, false);
    expect("six", {2, 3, 4, 5, 6, 12}, many, BIN_SMALL, true);
    expect("six, few products", {2, 3, 4, 5, 6, 12}, few, BIN_SMALL, false);
    expect("one", {5}, many, BIN_SMALL, false);
    numeric("after a spread pass", {5}, {1.0}, true, true);
    numeric("three heavy of six", {5, 6, 7, 11, 13, 14}, {.01, .01, .01, .6, .15, .22}, false, true);
    numeric("three rank kernels of seven, one with a fifteenth", {5, 6, 7, 8, 11, 13, 14},
            {.001, .001, .002, .002, .78, .068, .146}, false, true);
    numeric("three heavy hash kernels of six", {2, 3, 4, 5, 6, 13}, {.02, .02, .1, .1, .1, .66}, false, false);
    numeric("two heavy of six", {5, 6, 7, 11, 13, 14}, {.01, .01, .01, .02, .75, .2}, false, false);
    numeric("three heavy of five", {6, 7, 11, 13, 14}, {.02, .02, .6, .15, .21}, false, false);
    numeric("three heavy of five, and rows of one A entry", {1, 6, 7, 11, 13, 14}, {.02, .01, .01, .6, .15, .21}, false, false);
    return failed;
}
"""


def test_fork_rule(tmp_path):
    try:
        cc = hip_build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src, exe = tmp_path / "rule.hip", tmp_path / "rule"
    src.write_text(SOURCE)
    flags = [f for f in hip_build.flags() if f not in ("-fPIC", "-shared")]
    r = subprocess.run([cc] + flags + ["-I" + hip_build.CSRC, "-o", str(exe), str(src)], capture_output=True, text=True,
                       cwd=os.path.dirname(hip_build.CSRC))
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
