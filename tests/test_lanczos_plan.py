"""Host enumeration of the LDS that the one-workgroup Lanczos kernel touches.

The kernel (csrc/lanczos.hip) splits w = T q over chunks of a row; a thread
multiplies its LZ_TREG register columns with as many entries of q whether or
not its chunk is that long, zeros standing behind q.  An entry past those zeros
belongs to the work vector or to the partial sums, which other threads write
at that time and nothing has written in the first step: even with a factor of
zero a NaN there would reach the product.  The split and the layout live in a
header without HIP (csrc/launch_plan.hpp); here every index of every thread
is enumerated for every n of the kernel.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_14013_amd", "csrc")

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "launch_plan.hpp"
using namespace wc;
int main() {
    long checked = 0, bad = 0;
    for (int n = 1; n <= 640; ++n) {
        const LanczosPlan p = lanczos_plan(n);
        bool ok = p.nch >= 1 && p.w >= n + LZ_TREG && p.pp >= p.w + n && p.Q >= p.pp + (p.nch > 1 ? n * p.nch : 0);
        ok = ok && n * p.nch <= std::max(n, LZ_THREADS) && (p.nch == 1) == (n > LZ_THREADS / 2 || n <= LZ_CHUNK);
        // no chunk but the last shorter than half of LZ_CHUNK
        ok = ok && (p.nch == 1 || 2 * p.clen > LZ_CHUNK);
        std::vector<int> seen(n, 0);  // columns of row 0
        if (p.nch == 1) std::fill(seen.begin(), seen.end(), 1);
        for (int tid = 0; tid < LZ_THREADS && p.nch > 1; ++tid) {
            if (tid >= n * p.nch) break;
            const int cc = tid / n, cl0 = cc * p.clen, cl1 = std::min(n, cl0 + p.clen);
            ok = ok && cl0 < n;
            for (int u = 0; u < LZ_TREG; ++u) {
                ++checked;
                ok = ok && cl0 + u < n + LZ_TREG;  // q or its zeros
                if (tid % n == 0 && cl0 + u < cl1) ++seen[cl0 + u];
            }
            for (int l = cl0 + LZ_TREG; l < cl1; ++l)
                if (tid % n == 0) ++seen[l];
        }
        for (int s : seen) ok = ok && s == 1;
        if (!ok) { ++bad; printf("bad n %d: nch %d clen %d\n", n, p.nch, p.clen); }
    }
    printf("checked %ld bad %ld\n", checked, bad);
    return bad != 0;
}
"""


def test_lanczos_reads_stay_inside_the_vector_and_its_zeros(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "lz.cpp", tmp_path / "lz"
    src.write_text(DRIVER)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    assert int(r.stdout.split()[-3]) > 500_000
