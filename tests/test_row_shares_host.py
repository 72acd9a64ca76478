"""How the columns kernel of Winograd by axes deals the rows of a tile to its wavefronts: every row to one share, no operand read outside the
share's own rows.  The header is compiled for the host, as it is."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2002_12418_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "row_shares.hpp"
using namespace mnnconv;
int main()
{
    for (int A = 3; A <= 10; ++A)
        for (int Q = 2; Q <= 4; Q += 2) {
            if (A < Q) continue;
            const int steps = (A + Q - 1) / Q;
            int next = 0;
            for (int share = 0; share < Q; ++share) {
                const RowShare s = row_share(A, Q, share);
                if (s.first != next || s.rows < 1 || s.rows > steps) { std::printf("A=%d Q=%d share %d: rows %d + %d\n", A, Q, share, s.first, s.rows); return 1; }
                next = s.first + s.rows;
                for (int q = 0; q < steps; ++q) {
                    const int row = row_of_step(A, Q, share, q);
                    if (row < 0 || row >= s.rows || s.first + row >= A || (q < s.rows && row != q)) {
                        std::printf("A=%d Q=%d share %d step %d: reads row %d of %d\n", A, Q, share, q, s.first + row, A);
                        return 1;
                    }
                }
            }
            if (next != A) { std::printf("A=%d Q=%d: %d rows dealt\n", A, Q, next); return 1; }
        }
    return 0;
}
"""


def test_every_row_once_and_no_read_outside_a_share(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "shares.cpp", tmp_path / "shares"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
