"""The set-up work's host threads where memory runs out: every allocation of the
calling thread in turn fails.  The work is done, or the exception reaches the
caller; the process does not end.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_12011_amd", "csrc")

PROGRAM = r"""
#include "mdx_parallel.h"
#include <cstdio>
#include <cstdlib>
#include <new>
#include <stdexcept>

static thread_local long g_left = -1;   // allocations of this thread until one fails
void *operator new(std::size_t n)
{
    if (g_left >= 0 && g_left-- == 0) throw std::bad_alloc();
    if (void *p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main()
{
    int thrown = 0, whole = 0;
    for (long fail = 0; fail < 40; ++fail) {
        std::atomic<int> done[64] = {};
        bool out = false;
        g_left = fail;
        try {
            mdx::host::parallel_for(64, [&](int k) { done[k]++; });
        } catch (const std::bad_alloc &) {
            out = true;
        }
        g_left = -1;
        thrown += out;
        bool all = true;
        for (auto &d : done) all = all && d == 1;
        whole += all;
        if (!all && !out) return 1;
    }
    bool passed_on = false;   // an exception of the work itself
    try {
        mdx::host::parallel_for(64, [&](int k) { if (k == 7) throw std::runtime_error("7"); });
    } catch (const std::runtime_error &) {
        passed_on = true;
    }
    std::printf("thrown %d whole %d passed on %d\n", thrown, whole, passed_on);
    return passed_on && whole > 0 ? 0 : 2;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_allocations_that_fail(tmp_path):
    src, exe = tmp_path / "p.cpp", tmp_path / "p"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
