"""The fast-diagonalisation plane kernel multiplies whole MFMA steps: past the
end of a half it reads columns whose matrix entries are zero.  They have to lie
inside the row, where the staging has written every entry: beyond it is LDS that
another workgroup left, and zero times a NaN is a NaN.  The reads of every lane,
step and tile are enumerated on the host for all lengths the kernel serves."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2311_06926_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include "fd_layout.h"
// SPLIT: a tile that holds any value is read whole
template <typename T, bool SPLIT>
int check(const char* name) {
    int bad = 0;
    for (int nM = 2; nM <= 128; ++nM)
        for (int n = nM - 1; n <= nM; ++n) {  // directions of degree p and p - 1
            const int nt = ((nM + 1) / 2 + 15) / 16, he = (n + 1) / 2, ho = n / 2;
            const int ld = hp::plane_pitch<T>(n);
            int last = n - 1;
            for (int par = 0; par < 2; ++par) {
                const int h = par ? ho : he, off = par ? he : 0;
                for (int c = 0; c < nt; ++c) {
                    int steps = c + 1 < nt ? 4 : hp::mfma_steps<T>(h - 16 * c);
                    if (SPLIT && steps) steps = 4;
                    for (int lk = 0; lk < 4; ++lk)
                        for (int i = 0; i < steps; ++i) {
                            const int col = off + 16 * c + hp::mfma_row<T>(lk, i);
                            if (col > last) last = col;
                        }
                }
            }
            if (last >= ld || !(ld & 1)) {
                std::printf("%s nM=%d n=%d: column %d read, pitch %d\n", name, nM, n, last, ld);
                ++bad;
            }
        }
    return bad;
}
int main() {
    const int bad = check<double, false>("FP64") + check<float, false>("FP32") +
                    check<float, true>("split BF16");
    return bad != 0;
}
"""


def test_reads_stay_in_the_row(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text(SOURCE)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
