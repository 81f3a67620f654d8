"""Which form the entry-sampling products take (csrc/launch_plan.hpp).

F = G_w^T [Y0 Q, Y1 Q] joins the refinement's two vectors in one thin product of
2 r columns; past THIN_N columns the thin product declines, and one general
product of 2 r columns has too few tiles to fill the chip.  So the vectors are
joined only while their columns fit, which a host-compiled enumeration checks.

The latency-bound forms are taken where they are the faster ones: MEASURED
holds precond_apply (us, MI355X) in both forms at m = min(9 n r, 160000).
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_14013_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "launch_plan.hpp"
using namespace wc;
int main() {
    int bad = 0, joined = 0;
    for (int r = 1; r <= 64; ++r)
        for (int nv = 1; nv <= 2; ++nv) {
            const int per = thin_vectors(r, nv);
            // every vector once, and never a product too wide only because vectors were joined
            if (per < 1 || nv % per != 0 || (per > 1 && per * r > THIN_N)) { ++bad; printf("bad r %d nv %d: %d\n", r, nv, per); }
            joined += per == 2;
        }
    printf("joined %d bad %d\n", joined, bad);
    return bad != 0;
}
"""

SMALL = r"""
#include <cstdio>
#include <cstdlib>
#include "launch_plan.hpp"
int main(int argc, char** argv) {  // n r ...
    for (int i = 1; i + 1 < argc; i += 2) printf("%d\n", wc::entry_small(atoi(argv[i]), atoi(argv[i + 1])) ? 1 : 0);
}
"""

# n, r: latency-bound form, general form
MEASURED = {(100, 5): (65.6, 93.6), (100, 16): (117.4, 176.4), (300, 8): (110.2, 142.4), (400, 16): (244.4, 270.6),
            (512, 2): (56.2, 72.9), (512, 4): (70.2, 91.0), (512, 10): (182.2, 192.3), (512, 16): (298.0, 298.7),
            (640, 8): (173.2, 174.4), (768, 4): (91.7, 105.6), (768, 5): (147.3, 137.4), (768, 10): (261.9, 245.5),
            (900, 8): (246.9, 217.1), (1024, 2): (79.6, 81.6), (1024, 4): (110.9, 111.3), (1024, 5): (185.5, 150.6),
            (1024, 8): (269.4, 230.1), (1200, 4): (137.0, 128.4), (1500, 2): (104.3, 98.6), (1500, 5): (272.4, 209.1)}


def test_vectors_are_joined_only_while_the_thin_product_takes_them(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "e.cpp", tmp_path / "e"
    src.write_text(DRIVER)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert r.stdout.split()[1] == "8"


def test_latency_bound_forms_are_taken_where_they_are_faster(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "s.cpp", tmp_path / "s"
    src.write_text(SMALL)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    args = [str(v) for k in MEASURED for v in k]
    got = [int(v) for v in subprocess.run([str(exe), *args], capture_output=True, text=True, check=True).stdout.split()]
    assert len(got) == len(MEASURED)
    for (k, (small, general)), s in zip(MEASURED.items(), got):
        assert (small if s else general) <= 1.01 * min(small, general), k
    # H (n r doubles) and the partial sums (16 x EN_R x 16) in 160 KB of LDS
    pairs = [(n, r) for n in range(1, 1300) for r in range(1, 20)]
    got = [int(v) for i in range(0, len(pairs), 2000) for v in
           subprocess.run([str(exe), *(str(v) for k in pairs[i:i + 2000] for v in k)], capture_output=True, text=True,
                          check=True).stdout.split()]
    assert all(8 * (n * r + 16 * 16 * 16) <= 160 * 1024 and r <= 16 for (n, r), s in zip(pairs, got) if s)
