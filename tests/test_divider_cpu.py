"""The division by multiplication of the second pass (Divider in csrc/lnmod_launch.hpp) against the machine's own, over the
range it is used on: every divisor up to 5000, every power of two and its neighbours, 400 000 random ones; dividends at 0, at
the multiples of the divisor and just below them, at 2^31 - 1 and at random.  Needs only hipcc's host compiler."""
import os
import shutil
import subprocess

import pytest

from paper_2605_17923_amd import build

SOURCE = r"""
#include <cstdint>
#include <cstdio>
#include <random>
#include "lnmod_launch.hpp"
static long bad = 0;
static const uint32_t top = (1u << 31) - 1;
static void check(uint32_t d, uint32_t n) {
    if (n <= top && lnmod::Divider(d)(n) != n / d && bad++ < 5) std::printf("%u / %u = %u, got %u\n", n, d, n / d, lnmod::Divider(d)(n));
}
int main() {
    std::mt19937_64 r(1);
    auto all = [&](uint32_t d) {
        const uint32_t k = static_cast<uint32_t>(r() % (top / d + 1)) * d;
        for (const uint32_t n : {0u, d - 1, d, k, k - 1, top / d * d, top / d * d - 1, top, static_cast<uint32_t>(r() & top)}) check(d, n);
    };
    for (uint32_t d = 1; d <= 5000; ++d) all(d);
    for (int s = 0; s < 31; ++s)
        for (int e = -1; e <= 1; ++e)
            if ((int64_t{1} << s) + e >= 1) all((1u << s) + e);
    for (int i = 0; i < 400000; ++i) all(static_cast<uint32_t>((r() & top) >> (r() % 31)) | 1u);
    for (int i = 0; i < 400000; ++i) all((static_cast<uint32_t>((r() & top) >> (r() % 31)) | 1u) + 1u);
    std::printf("%ld wrong\n", bad);
    return bad != 0;
}
"""


def test_division_by_multiplication(tmp_path):
    hipcc = build._hipcc()
    if shutil.which(hipcc) is None and not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    src, exe = str(tmp_path / "divider.cpp"), str(tmp_path / "divider")
    with open(src, "w") as f:
        f.write(SOURCE)
    res = subprocess.run([hipcc, "-std=c++17", "-O1", "-I", build.CSRC, "-I", build.INCLUDE, src, "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.endswith("0 wrong\n"), res.stdout
