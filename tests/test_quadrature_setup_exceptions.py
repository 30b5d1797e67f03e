"""No C++ exception crosses the C interface: when the host runs out of memory
while the quadrature operator's point tables are made, quad_setup returns an
error and leaves an empty operator that can be set up again."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2311_06926_amd")

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <new>
#include "hp_internal.h"

static long allowed = -1;  // allocations until the next fails (-1: no limit)
void* operator new(std::size_t n) {
    if (allowed == 0) throw std::bad_alloc();
    if (allowed > 0) --allowed;
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
    hp_ctx c;
    c.tab = hp::build_tables(5, 3, 12.5);
    c.E = 5;
    c.p = 3;
    c.nN = c.tab.nN;
    c.nM = 7;
    c.opts.max_rhs = 1;
    for (int n = 0; n < 4; ++n) {
        hp::QuadOp q;
        hipError_t e;
        allowed = n;
        try {
            e = hp::quad_setup(&c, &q);
        } catch (...) {
            std::printf("an exception left quad_setup (%d allocations)\n", n);
            return 1;
        }
        allowed = -1;
        if (e != hipErrorOutOfMemory || q.ready || q.tables || q.scratch) {
            std::printf("status %d after %d allocations\n", (int)e, n);
            return 1;
        }
    }
    return 0;
}
"""


def test_out_of_host_memory(tmp_path):
    cxx = shutil.which("g++")
    lib = os.path.join(PKG, "libhyperpower.so")
    rocm = "/opt/rocm"
    if not cxx or not os.path.exists(lib) or not os.path.isdir(rocm):
        pytest.skip("no host compiler or library")
    src, exe = tmp_path / "setup.cpp", tmp_path / "setup"
    src.write_text(SOURCE)
    subprocess.run([cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", f"{rocm}/include",
                    "-I", os.path.join(PKG, "csrc"), str(src), "-o", str(exe), lib,
                    f"-Wl,-rpath,{PKG}", f"-L{rocm}/lib", f"-Wl,-rpath,{rocm}/lib", "-lamdhip64"],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
