"""The device functions of mt_math.h, compiled for the host: the same polynomials and
fused operations in the same order, with the two hardware instructions that they
start from (reciprocal estimate, exponent and mantissa) written out here.

Bounds: those the header states, 0.9 units in the last place for 2^x (its Horner
sum rounds near 1 and f q(f) reaches 0.41), 0.6 for log2 and 1/x (the last rounding and
1/10 more), 1.2e-10 for the float path's 2^x.  Exact values: long double, whose functions
are good to about 2^-10 units of a double.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <cmath>
#define __device__
#define __forceinline__ inline
static double g_est;       // relative error of the reciprocal estimate
static float __builtin_amdgcn_exp2f(float x) { return exp2f(x); }
static float __builtin_amdgcn_logf(float x) { return log2f(x); }
static float __builtin_amdgcn_rcpf(float x) { return 1.f / x; }
static double __builtin_amdgcn_rcp(double x) { return (1.0 / x) * (1.0 + g_est); }
static double __builtin_amdgcn_ldexp(double x, int e) { return ldexp(x, e); }
static double __builtin_amdgcn_frexp_mant(double x) { int e; return frexp(x, &e); }
static int __builtin_amdgcn_frexp_exp(double x) { int e = 0; frexp(x, &e); return e; }
#include "mt_math.h"
extern "C" void apply(int f, long n, double est, const double* x, double* y) {
    g_est = est;
    for (long i = 0; i < n; ++i)
        y[i] = f == 0 ? mt::dexp2(x[i]) : f == 1 ? mt::dlog2<true>(x[i]) : f == 2 ? mt::drcp(x[i]) : f == 3 ? mt::exp2_acc(x[i])
                                                              : mt::drcp_inf(x[i]);
}
"""


@pytest.fixture(scope="module")
def apply(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("math")
    (d / "m.cpp").write_text(SHIM)
    subprocess.run([gxx, "-O1", "-std=c++17", "-mfma", "-ffp-contract=off", "-fno-builtin", "-shared", "-fPIC",
                    "-I" + os.path.join(ROOT, "paper_1909_11474_amd", "csrc"), str(d / "m.cpp"), "-o",
                    str(d / "m.so")], check=True, capture_output=True)
    lib = ctypes.CDLL(str(d / "m.so"))
    p = ctypes.c_void_p

    def run(f, x, est=0.0):
        x = np.ascontiguousarray(x, dtype=np.float64)
        y = np.empty_like(x)
        lib.apply(ctypes.c_int(f), ctypes.c_long(x.size), ctypes.c_double(est), p(x.ctypes.data), p(y.ctypes.data))
        return y

    return run


def ulps(got, exact):
    return float((np.abs(got.astype(np.longdouble) - exact) / np.spacing(np.abs(exact.astype(np.float64)))).max())


g = np.random.Generator(np.random.PCG64(1))
EXP_ARGS = np.concatenate([g.uniform(-1020, 1020, 200000), g.uniform(-2, 2, 200000),
                           np.rint(g.uniform(-60, 60, 50000)) + 0.5 + g.uniform(-1e-9, 1e-9, 50000),
                           g.choice([-1, 1], 50000) * 10.0 ** g.uniform(-18, 0, 50000), [0.0, 1.0, -1.0, -0.477]])
LOG_ARGS = np.concatenate([10.0 ** g.uniform(-300, 300, 200000), g.uniform(0.4, 3.0, 200000),
                           1.0 + g.choice([-1, 1], 100000) * 10.0 ** g.uniform(-15, -1, 100000),
                           np.sqrt(0.5) * (1.0 + g.uniform(-1e-9, 1e-9, 50000)),
                           np.sqrt(2.0) * (1.0 + g.uniform(-1e-9, 1e-9, 50000)),
                           [np.nextafter(1, 0), np.nextafter(1, 2), 2.0, 0.5, 5e-324, 1.7976931348623157e308]])


@pytest.mark.parametrize("est", [0.0, 2.0 ** -23, -2.0 ** -23])
def test_errors_in_units_of_the_last_place(apply, est):
    assert ulps(apply(0, EXP_ARGS), np.exp2(EXP_ARGS.astype(np.longdouble))) <= 0.9
    assert ulps(apply(1, LOG_ARGS, est), np.log2(LOG_ARGS.astype(np.longdouble))) <= 0.6
    x = np.concatenate([10.0 ** g.uniform(-307, 307, 200000), g.uniform(1, 2, 200000)])
    x = np.concatenate([x, -x])
    assert ulps(apply(2, x, est), 1 / x.astype(np.longdouble)) <= 0.6
    a = EXP_ARGS[np.abs(EXP_ARGS) < 1000]
    exact = np.exp2(a.astype(np.longdouble))
    assert np.abs(apply(3, a) / exact - 1).max() <= 1.2e-10


def test_ends_of_the_range(apply):
    inf = np.inf
    assert np.array_equal(apply(4, [inf, 1e300, 2.0]), [0.0, 1e-300, 0.5])
    assert apply(1, [inf])[0] == inf and apply(1, [1.0])[0] == 0.0
    # (infinite arguments of 2^x need the device's saturating conversion to int)
    assert np.array_equal(apply(0, [1e9, 1024.0, -1e9, -1100.0]), [inf, inf, 0.0, 0.0])
    for f in (0, 1, 2, 4):
        assert np.isnan(apply(f, [np.nan])[0])
