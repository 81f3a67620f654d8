"""The batched staging's host threads (csrc/host_pool.hpp) when one cannot be started.

Starting a thread may fail for want of threads (std::system_error) or of memory
(std::bad_alloc).  With others already running, an exception that left the
function then would end the process: their std::thread objects would be
destroyed unjoined.  Here every allocation of a start fails in turn, and so does
the reservation before them; the work must be done all the same.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_14013_amd", "csrc")

DRIVER = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include "host_pool.hpp"
thread_local int allowed = -1;  // allocations of this thread before one fails (-1: all succeed)
void* operator new(std::size_t n) {
    if (allowed == 0) { allowed = -1; throw std::bad_alloc(); }
    if (allowed > 0) --allowed;
    return std::malloc(n);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
int main() {
    int bad = 0;
    for (int fail = -1; fail < 8; ++fail)
        for (int extra : {-1, 0, 1, 7}) {
            std::atomic<int> next{0}, done{0};
            auto work = [&] {
                while (next++ < 100) ++done;
            };
            allowed = fail;
            wc::run_shared(extra, work);
            allowed = -1;
            bad += done != 100;
        }
    std::printf("bad %d\n", bad);
    return bad != 0;
}
"""


def test_work_is_done_when_a_thread_cannot_be_started(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "p.cpp", tmp_path / "p"
    src.write_text(DRIVER)
    subprocess.run([cxx, "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
