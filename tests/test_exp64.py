"""The fp64 exponentials of the accept pass (csrc/exp64.h), compiled for the host with the device's words defined away:
relative error against 80-bit long doubles, and the ends of the range."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_20330_amd", "csrc")

# The constant form of fma is one instruction of the device; here it is fma.
SHIM = r"""
#include <cmath>
#include <cstring>
using std::fma; using std::fmax; using std::fmin; using std::rint; using std::ldexp; using std::fabs;
#define __device__
#define __forceinline__ inline
#define asm(...) d = fma(a, b, k)
static inline long long __double_as_longlong(double x) { long long v; std::memcpy(&v, &x, 8); return v; }
static inline bool __any(bool x) { return x; }
#include "exp64.h"
extern "C" void exp64(int which, const double* x, double* y, int n)
{
    for (int i = 0; i < n; ++i) y[i] = which == 0 ? exp_c(x[i]) : which == 1 ? exp_tab(x[i], kExp2Table) : exp_shift(x[i], kExp2Table);
}
"""


@pytest.fixture(scope="module")
def exp64(tmp_path_factory):
    d = tmp_path_factory.mktemp("exp64")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o",
                    str(d / "exp64.so")], check=True)
    lib = ctypes.CDLL(str(d / "exp64.so"))

    def call(which, x):
        x = np.ascontiguousarray(x, dtype=np.float64)
        y = np.empty_like(x)
        lib.exp64(which, x.ctypes.data_as(ctypes.c_void_p), y.ctypes.data_as(ctypes.c_void_p), len(x))
        return y
    return call


@pytest.mark.parametrize("which", [0, 1, 2])
def test_ends_of_the_range(exp64, which):
    """+inf from overflow on, however large the argument (a shift eta (q - p) may be of any size); 0 far below, for -inf and NaN."""
    big = np.array([710.0, 800.0, 1e4, 2.3e7, 2.4e7, 3e7, 4.7e7, 9.3e7, 1e8, 1e9])
    assert np.all(np.isposinf(exp64(which, big))), exp64(which, big)
    assert not exp64(which, np.array([-746.0, -1e5, -1e30, -np.inf, np.nan])).any()
    assert np.all(exp64(which, np.array([0.0, -0.0])) == 1.0)
    if which:                                                  # (the exponential of the decisions sees no such arguments)
        assert np.all(np.isposinf(exp64(which, np.array([1e15, 1e30, 3e38, np.inf]))))


@pytest.mark.parametrize("which", [0, 1, 2])
@pytest.mark.parametrize("lo,hi", [(-2.0 ** -6, 2.0 ** -6), (-1.0, 0.0), (-30.0, 0.0), (-700.0, 0.0), (-20.0, 20.0), (0.0, 700.0)])
def test_relative_error(exp64, which, lo, hi):
    """All three forms stay within 1.4e-16: half a unit of the last place (1.11e-16) for the final rounding, the rest for the
    polynomial and the reduction.  What the draw computes with the table is no coarser than what the decisions use."""
    x = np.random.default_rng(int(which + 10 * (hi - lo))).uniform(lo, hi, 400000)
    want = np.exp(x.astype(np.longdouble))                     # 64 bits of mantissa: 2^-63 of its own
    assert np.finfo(np.longdouble).nmant >= 63
    err = np.abs((exp64(which, x).astype(np.longdouble) - want) / want).max()
    assert float(err) <= 1.4e-16, float(err)
