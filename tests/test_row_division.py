"""The product-and-shift division of the row map (csrc/fwd_shape.h) is exact for every number below 2^31: quotients change at the
multiples of the divisor only, so those and their neighbours are compared, from both ends and at random."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_09237_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <random>
#include "fwd_shape.h"
int main() {
    std::mt19937 g(1);
    long n = 0, wrong = 0;
    auto check = [&](uint32_t d) {
        const RowDiv r = row_div((int32_t)d);
        const uint32_t top = 0x7fffffffu, last = top / d;
        auto at = [&](uint32_t m) { ++n; wrong += r.quotient(m) != m / d; };
        for (uint32_t i = 0; i < 200; ++i) {
            const uint32_t k = i < 50 ? (i < last ? i : last) : i < 100 ? (last > i - 50 ? last - (i - 50) : 0) : g() % ((uint64_t)last + 1);
            at(k * d);
            if (k) at(k * d - 1);
            if ((uint64_t)k * d + d - 1 <= top) at(k * d + d - 1);
        }
        at(0); at(top); at(top - 1);
    };
    for (uint32_t d = 1; d < 5000; ++d) check(d);
    for (int s = 1; s < 31; ++s) for (int e = -2; e <= 2; ++e) if ((1ll << s) + e > 0) check((1u << s) + e);
    check(0x7fffffffu);
    for (int i = 0; i < 20000; ++i) check(1 + g() % 0x7ffffffeu);
    printf("numbers %ld wrong %ld\n", n, wrong);
    return wrong ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_row_division_is_exact(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
