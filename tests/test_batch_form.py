"""The batched solver's pass settings without a tuning (csrc/launch_plan.hpp).

MEASURED holds four iterations of 32 instances (ms, MI355X, FP64 and FP32 inner
solves) with 4 rows per wave and 16 x 16 tiles and with 2 rows and 32 x 32; the rule
has to take one that is no more than 4% slower than the other.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_14013_amd", "csrc")

MEASURED = {16: ((26.3, 27.1), (39.0, 41.4)), 24: ((35.8, 37.0), (50.4, 54.3)), 28: ((33.1, 33.8), (41.9, 44.3)),
            30: ((33.5, 33.8), (42.1, 44.2)), 32: ((38.1, 39.5), (40.2, 41.8)), 33: ((46.9, 45.8), (47.0, 47.6)),
            35: ((48.1, 46.3), (48.4, 48.2)), 36: ((51.1, 48.4), (50.1, 49.8)), 40: ((53.6, 47.8), (50.1, 49.9)),
            44: ((60.2, 54.7), (57.0, 55.9)), 47: ((81.2, 75.7), (78.4, 78.0)), 48: ((77.4, 72.2), (74.9, 75.2)),
            56: ((104.3, 96.8), (96.3, 95.1)), 72: ((208.4, 189.1), (183.6, 178.2)), 128: ((840.6, 798.4), (778.4, 747.2))}


def test_rule_agrees_with_the_measurements(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "b.cpp", tmp_path / "b"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "launch_plan.hpp"\n'
                   'int main(int argc, char** argv) { for (int i = 1; i < argc; ++i) { const wc::BatchForm f = '
                   'wc::batch_form(atoi(argv[i])); printf("%d %d\\n", f.rows_per_wave, f.gemm_tile); } }\n')
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), *map(str, MEASURED)], capture_output=True, text=True, check=True)
    for n, line in zip(MEASURED, r.stdout.splitlines()):
        form = [(4, 16), (2, 32)].index(tuple(map(int, line.split())))
        for times in MEASURED[n]:
            assert times[form] <= 1.04 * min(times), n
