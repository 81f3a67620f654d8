"""Which product each of the entry-sampling products takes (csrc/launch_plan.hpp).

F = G_w^T [Y0 Q, Y1 Q] joins the refinement's two vectors in one thin product of
2 r columns; past THIN_N columns the thin product declines, and one general
product of 2 r columns has too few tiles to fill the chip.  So the vectors are
joined only while their columns fit, which a host-compiled enumeration checks.
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
