"""Which form the dense rows' operator takes (csrc/launch_plan.hpp).

MEASURED holds newton_apply (us, MI355X) with the off-diagonal blocks from the
explicit script-A script-Q and as products with G_w; the rule has to take one
that is no more than 5% slower than the other.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_14013_amd", "csrc")

# n, r, m: explicit, products
MEASURED = {(32, 3, 288): (13.8, 44.5), (64, 30, 1664): (43.2, 78.3), (100, 10, 3000): (64.8, 122.0),
            (100, 30, 4040): (97.1, 113.2), (100, 60, 4040): (115.7, 123.6), (150, 10, 4500): (173.7, 227.6),
            (150, 20, 9000): (347.1, 322.2), (150, 30, 9060): (381.5, 326.9), (150, 60, 9060): (456.0, 328.3),
            (200, 3, 1800): (128.7, 156.7), (200, 10, 6000): (358.1, 402.1), (200, 15, 9000): (545.4, 570.6),
            (200, 20, 12000): (773.1, 679.5), (200, 30, 16080): (1103.3, 886.4), (200, 60, 16080): (1301.8, 900.4),
            (300, 5, 4500): (603.0, 652.8), (300, 10, 9000): (1152.8, 1119.2), (300, 20, 18000): (2349.2, 2126.8),
            (200, 100, 300): (77.7, 123.0), (200, 40, 4000): (307.6, 269.3), (300, 50, 1000): (181.8, 199.8)}


def test_rule_agrees_with_the_measurements(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "d.cpp", tmp_path / "d"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "launch_plan.hpp"\n'
                   'int main(int argc, char** argv) { for (int i = 1; i + 1 < argc; i += 2) '
                   'printf("%d\\n", wc::dense_explicit(atol(argv[i]), atol(argv[i + 1])) ? 1 : 0); }\n')
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    args = [str(v) for n, r, m in MEASURED for v in (m, n * r - r * (r - 1) // 2)]
    got = [int(v) for v in subprocess.run([str(exe), *args], capture_output=True, text=True, check=True).stdout.split()]
    assert len(got) == len(MEASURED)
    for (k, (explicit, products)), e in zip(MEASURED.items(), got):
        assert (explicit if e else products) <= 1.05 * min(explicit, products), k
