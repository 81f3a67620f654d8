"""The Sturm test of the Lanczos tridiagonal (csrc/sturm.hpp) against eigvalsh.

The header is free of HIP: the kernel's stopping test, the host's bisection and
this test share the recurrence.  Its pivots are backward stable: each is exact
for entries changed by a few units in the last place, so the answer is right
at every point further than that, times the norm, from the smallest eigenvalue.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_14013_amd", "csrc")
EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def below(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("sturm")
    (d / "s.cpp").write_text('#include "sturm.hpp"\n'
                             'extern "C" int below(const double* a, const double* b, int k, double x) '
                             '{ return wc::eigenvalue_below(a, b, k, x); }\n')
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "s.cpp"), "-o", str(d / "s.so")],
                   check=True)
    f = ctypes.CDLL(str(d / "s.so")).below
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_double]

    def call(a, b, x):
        a, b = (np.ascontiguousarray(v, dtype=np.float64) for v in (a, b))
        return bool(f(a.ctypes.data, b.ctypes.data, len(a), x))

    return call


def smallest(a, b):
    return np.linalg.eigvalsh(np.diag(a) + np.diag(b, 1) + np.diag(b, -1))[0]


@pytest.mark.parametrize("k", [1, 2, 3, 17, 64])
def test_answer_next_to_the_eigenvalue(below, k):
    # eigvalsh itself is off by a few EPS times the norm
    rng = np.random.default_rng(k)
    for _ in range(50):
        a, b = rng.standard_normal(k), rng.standard_normal(k - 1)
        lam, norm = smallest(a, b), np.abs(a).max() + 2.0 * np.abs(np.r_[b, 0.0]).max()
        d = 2 * (k + 10) * EPS * norm
        assert below(a, b, lam + d) and not below(a, b, lam - d)


@pytest.mark.parametrize("scale", [1e-150, 1.0, 1.5e4, 1e8, 1e150])
def test_zero_and_overflowing_pivots(below, scale):
    for k in (2, 4, 64):
        b = scale * np.linspace(1.0, 2.0, k - 1)
        assert below(np.zeros(k), b, 0.0)  # the first pivot is zero
        a = np.r_[1e-300, np.zeros(k - 1)]
        assert below(a, b, 0.0)  # the second is -infinity where b^2 is large
    assert below([0.0], [], 0.0) and not below([scale], [], 0.0)
