"""Division by constants the host knows: exact for every dividend below 2^31.  The header's arithmetic is compiled for the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2002_12418_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#define __device__
#define __forceinline__ inline
static unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)(((unsigned long long)a * b) >> 32); }
#include "fast_div.hpp"
using namespace mnnconv;
int main()
{
    unsigned long long rng = 12418;
    auto next = [&] { rng = rng * 6364136223846793005ull + 1442695040888963407ull; return (unsigned)(rng >> 33); };      // below 2^31
    for (unsigned i = 0; i < 60000; ++i) {
        const unsigned d = i < 20000 ? i + 1 : i < 20031 ? 1u << (i - 20000) : i < 20062 ? (1u << (i - 20031)) + 1 : i < 20093 ? (2u << (i - 20062)) - 1 : next() >> next() % 31;
        if (d < 1 || d >= 1u << 31) continue;
        const ConstDiv c = make_constdiv(d);
        const FastDiv f = make_fastdiv(d);
        for (unsigned j = 0; j < 200; ++j) {
            const unsigned m = next() >> next() % 31, q = m / d;
            const unsigned n = j % 4 == 0 ? m : j % 4 == 1 ? q * d : j % 4 == 2 ? (q ? q * d - 1 : 0) : j == 3 ? 0x7FFFFFFFu : 0x7FFFFFFFu - next() % d;
            if (const_div(n, c) != n / d || fast_div(n, f) != n / d) { std::printf("%u / %u\n", n, d); return 1; }
        }
    }
    return 0;
}
"""


def test_exact_below_two_to_the_31(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("")
    (tmp_path / "div.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", str(tmp_path), "-I", CSRC, str(tmp_path / "div.cpp"), "-o", str(tmp_path / "div")], check=True, timeout=120)
    r = subprocess.run([str(tmp_path / "div")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
