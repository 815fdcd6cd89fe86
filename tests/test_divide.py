"""The divisions that the kernels' index arithmetic stands on (csrc/divide.h), with the host's compiler: both forms against the
processor's division over the numerators that they are said to serve."""
import subprocess

import pytest

from paper_2006_09791_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "divide.h"
using namespace gspc;

int main(int, char **a) {
    const unsigned d = (unsigned)std::strtoull(a[1], nullptr, 10), m = div_magic(d);
    const unsigned long long top = (1ull << 32) / d;      // fast_div: (n + 1) * d <= 2^32
    unsigned long long bad = 0;
    auto check = [&](unsigned long long n) {
        if (n > 0xfffffffeull) return;
        const unsigned q = (unsigned)n / d, f = fast_div((unsigned)n, m);
        bad += n < top ? f != q : f != q && f + 1 != q;   // beyond: at most one too low
        bad += fast_div_any((unsigned)n, d, m) != q;
    };
    for (unsigned long long n = 0; n < 70000; ++n) check(n), check(top - 35000 + n), check(0xfffffffeull - n);
    for (unsigned long long k = 0, step = (1ull << 32) / d / 9973 + 1; k * d <= 0xffffffffull; k += step)   // around the multiples
        check(k * d), check(k * d + d - 1), check(k * d + 1), check(k * d + d / 2);
    std::printf("%llu\n", bad);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("divide")
    (d / "divide.cpp").write_text(PROGRAM)
    exe = str(d / "divide")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", build.CSRC, str(d / "divide.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("d", [1, 2, 3, 7, 9, 14, 16, 49, 196, 255, 256, 257, 641, 4096, 12544, 50176, 65535, 65536, 65537, 999983,
                               2 ** 24 + 1, 2 ** 31 - 1, 2 ** 31, 2 ** 32 - 1])
def test_divisions_by_reciprocals(program, d):
    assert subprocess.run([program, str(d)], check=True, capture_output=True, text=True).stdout.strip() == "0"
