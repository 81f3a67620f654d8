"""How far ahead the 64 x 64 FP64 product issues its loads (csrc/launch_plan.hpp).

MEASURED holds C -= op(A) op(B) (us, MI355X) two K steps ahead and one; the rule has
to take one that is no more than 4% slower than the other, and one step ahead
only for A B^T, the one product that is built in that form.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_14013_amd", "csrc")

# ta, tb, m = n, k: two steps, one
MEASURED = {(0, 1, 500, 500): (37.8, 39.8), (0, 1, 1000, 1000): (68.9, 72.9), (0, 1, 1500, 1500): (199.5, 207.6),
            (0, 1, 1700, 1700): (227.3, 237.0), (0, 1, 1750, 1750): (321.3, 301.1), (0, 1, 1800, 1800): (329.6, 309.6),
            (0, 1, 2000, 2000): (357.4, 335.8), (0, 1, 2000, 100): (37.9, 32.6), (0, 1, 1900, 256): (56.1, 53.2),
            (0, 1, 2100, 2100): (457.9, 462.4), (0, 1, 2500, 2500): (755.1, 735.0), (0, 1, 3000, 3000): (1142.8, 1124.0),
            (0, 1, 4000, 4000): (2464.3, 2530.0), (0, 1, 5000, 256): (283.8, 286.8), (0, 1, 1792, 1792): (281.8, 285.6),
            (0, 1, 2048, 2048): (322.3, 327.5), (0, 1, 3200, 3200): (1172.4, 1238.4), (1, 0, 1000, 1000): (60.6, 69.2),
            (1, 0, 1750, 1750): (295.3, 293.4), (1, 0, 2000, 2000): (325.6, 326.5), (1, 0, 3000, 3000): (1056.9, 1120.7)}


def test_rule_agrees_with_the_measurements(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "g.cpp", tmp_path / "g"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "launch_plan.hpp"\n'
                   'int main(int argc, char** argv) { for (int i = 1; i + 3 < argc; i += 4) printf("%d\\n", '
                   'wc::two_steps_ahead(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atol(argv[i + 3])) ? 1 : 0); }\n')
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def rule(args):
        flat = [str(int(v)) for a in args for v in a]
        r = subprocess.run([str(exe), *flat], capture_output=True, text=True, check=True)
        return [int(v) for v in r.stdout.split()]

    two = rule([(ta, tb, n % 64 != 0 or k % 16 != 0, (-(-n // 64)) ** 2) for ta, tb, n, k in MEASURED])
    for (k, (t2, t1)), t in zip(MEASURED.items(), two):
        assert (t2 if t else t1) <= 1.04 * min(t2, t1), k
    others = [(ta, tb, e, w) for ta, tb in ((0, 0), (1, 0), (1, 1)) for e in (0, 1) for w in (1, 700, 800, 2000, 9000)]
    assert all(rule(others))
