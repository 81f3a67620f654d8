"""The batched solver's factorisations leave a bad pivot through a barrier.

wg_potrf and wg_spd_inverse (csrc/batched.hip) are run here by host threads: the
functions' own source is compiled with the host compiler, `gd` being a number
whose reads can be held up and bsync() a barrier with a time limit.  The second
wave is held at its read of the bad pivot until the first wave has come back
from the call and refilled the matrix, as guard_step does, or has had time to.
Were the return not preceded by a barrier, the second wave would find a good
pivot and go on to barriers that nobody else reaches.
"""
import os
import re
import shutil
import subprocess

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_14013_amd", "csrc",
                   "batched.hip")

HEAD = r"""
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <thread>
#include <vector>
#define __device__
#define __noinline__
using std::min;
constexpr int BT = 128, BWV = BT / 64;
struct Idx { int x; };
thread_local Idx threadIdx;

std::mutex mu;
std::condition_variable cv;
int waiting = 0, phase = 0;
void bsync() {
    std::unique_lock<std::mutex> l(mu);
    const int p = phase;
    if (++waiting == BT) {
        waiting = 0;
        ++phase;
        cv.notify_all();
    } else if (!cv.wait_for(l, std::chrono::seconds(20), [&] { return phase != p; })) {
        printf("a barrier that not all threads reach\n");
        fflush(stdout);
        _Exit(1);
    }
}

std::atomic<bool> refilled{false};
struct gd {
    double v = 0.0;
    operator double() const {
        if (v == -7.0 && threadIdx.x >= 64)  // the bad pivot
            for (int t = 0; t < 20 && !refilled; ++t) std::this_thread::sleep_for(std::chrono::milliseconds(5));
        return v;
    }
    gd& operator=(double x) { v = x; return *this; }
    gd& operator=(const gd& x) { return *this = static_cast<double>(x); }
    gd& operator/=(double x) { v /= x; return *this; }
    gd& operator-=(double x) { v -= x; return *this; }
};
"""

MAIN = r"""
int main() {
    constexpr int n = 5;
    std::vector<gd> A(n * n), colk(n);
    int bad = 0;
    for (int which = 0; which < 2; ++which)
        for (int j = 0; j < n; ++j) {
            for (auto& a : A) a.v = 0.0;
            for (int i = 0; i < n; ++i) A[i + n * i].v = i == j ? -7.0 : 4.0;
            refilled = false;
            std::vector<int> got(BT);
            std::vector<std::thread> ts;
            for (int t = 0; t < BT; ++t)
                ts.emplace_back([&, t] {
                    threadIdx.x = t;
                    got[t] = which == 0 ? wg_potrf(n, A.data(), n) : wg_spd_inverse(n, A.data(), n, colk.data());
                    if (t == 0) {
                        for (int i = 0; i < n; ++i) A[i + n * i].v = 1.0;
                        refilled = true;
                    }
                });
            for (auto& t : ts) t.join();
            for (int g : got) bad += g != j + 1;
        }
    printf("wrong returns: %d\n", bad);
    return bad != 0;
}
"""


def test_bad_pivots_return_through_a_barrier(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    text = open(SRC).read()
    fns = [re.search(r"__device__ __noinline__ int " + f + r"\(.*?\n}\n", text, re.S).group(0)
           for f in ("wg_potrf", "wg_spd_inverse")]
    src, exe = tmp_path / "b.cpp", tmp_path / "b"
    src.write_text(HEAD + "\n".join(fns) + MAIN)
    subprocess.run([cxx, "-std=c++17", "-O1", "-pthread", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
