"""The FP64 elementary functions of the kernels (csrc/gm_math.h), compiled for
the host with the hardware estimates replaced by values rounded to FP32, against
the 80-bit library.

Bars in units in the last place: one half for the last rounding, plus the
roundings of the terms added to the leading one.  log, log2: about four
roundings (2^-53 relative, up to one unit) of a term at most 1 % of the result,
0.04 to 0.08.  sin, cos: three roundings of the cubic term, 0.0807 at |f| = 1/4
where the result is in [1/2, 1): 0.24.  sqrt: a correctly rounded remainder
step.  rcp: two Newton steps; rsq: its correction is a product of rounded
factors, one unit.  The HIP library's own are 0.69, 0.64, 0.87, 0.5, 0.5, 1.49."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_12273_amd", "csrc")
LD = np.longdouble

HOST = r"""
#include <cmath>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_frexp_mant(x) ([](double v) { int e; return std::frexp(v, &e); }(x))
#define __builtin_amdgcn_frexp_exp(x) ([](double v) { int e; std::frexp(v, &e); return e; }(x))
static double rcp_est(double x) { int e; const double m = std::frexp(x, &e); return std::ldexp((double)(float)(1.0 / m), -e); }
static double rsq_est(double x)
{
    int e;
    double m = std::frexp(x, &e);
    if (e & 1) { m *= 2; --e; }
    return std::ldexp((double)(float)(1.0 / std::sqrt(m)), -e / 2);
}
#define __builtin_amdgcn_rcp rcp_est
#define __builtin_amdgcn_rsq rsq_est
using std::fma;
#include "gm_math.h"
#define EACH(name) extern "C" void t_##name(const double* x, double* y, long n) { for (long i = 0; i < n; ++i) y[i] = gm::name(x[i]); }
EACH(rcp64) EACH(rsq64) EACH(log2_64) EACH(log_64) EACH(sqrt_64)
extern "C" void t_sincospi(const double* x, double* s, double* c, long n) { for (long i = 0; i < n; ++i) gm::sincospi_64(x[i], s[i], c[i]); }
extern "C" double t_new_rho(const double* s, const double* t, const double* rh, double omega, long n)
{
    gm::Sum2 q[2] = {};
    for (long i = 0; i < n; ++i) {
        gm::mul_add2(q[0], rh[i], s[i]);
        gm::mul_add2(q[1], rh[i], t[i]);
    }
    return gm::value2(gm::sub_scaled2(q[0], omega, q[1]));
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or np.finfo(LD).nmant < 63:
        pytest.skip("needs g++ and an 80-bit long double")
    d = tmp_path_factory.mktemp("math")
    (d / "host.cpp").write_text(HOST)
    so = str(d / "libmath.so")
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-ffp-contract=off", "-w", "-I", CSRC,
                    str(d / "host.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


def _call(lib, name, x, outs=1):
    x = np.ascontiguousarray(x)
    y = [np.empty_like(x) for _ in range(outs)]
    p = [ctypes.c_void_p(a.ctypes.data) for a in [x] + y]
    getattr(lib, "t_" + name)(*p, ctypes.c_long(x.size))
    return y[0] if outs == 1 else y


def _ulps(got, ref):
    ok = ref != 0
    _, e = np.frexp(ref[ok])
    return float(np.max(np.abs(got[ok].astype(LD) - ref[ok]) / np.ldexp(LD(1), e - 53)))


def _wide(rng, n, lo, hi):
    return np.exp(rng.uniform(lo, hi, n))


@pytest.mark.parametrize("name,ref,bar", [
    ("log2_64", np.log2, 0.6), ("log_64", np.log, 0.6), ("sqrt_64", np.sqrt, 0.501),
    ("rcp64", lambda x: 1 / x, 0.51), ("rsq64", lambda x: 1 / np.sqrt(x), 1.01)])
def test_one_argument_functions(lib, name, ref, bar):
    rng = np.random.default_rng(7)
    n = 400000
    sets = [1.0 - rng.random(n), _wide(rng, n, -36, 0), np.array([2.0 ** -53, 0.5, 1.0, np.nextafter(1.0, 0)])]
    if name != "log_64":  # arguments above one too
        sets += [rng.uniform(0.25, 1.75, n), _wide(rng, n, -500, 500), np.array([2.0, np.nextafter(1.0, 2), 1e300])]
    for x in sets:
        assert _ulps(_call(lib, name, x), ref(x.astype(LD))) <= bar


def test_sine_and_cosine(lib):  # of multiples of 2^-52 in [0, 2), twice the uniform draws
    rng = np.random.default_rng(8)
    a = np.concatenate([2.0 * rng.random(1000000), np.arange(8) / 4.0, np.nextafter(np.arange(1, 9) / 4.0, 0),
                        np.nextafter(np.arange(1, 8) / 4.0, 2), 2.0 ** -np.arange(1.0, 53.0)])
    s, c = _call(lib, "sincospi", a, 2)
    q = np.rint(2 * a).astype(np.int64)
    f = a.astype(LD) - q.astype(LD) / 2
    pi = 4 * np.arctan(LD(1))
    s0, c0 = np.sin(pi * f), np.cos(pi * f)
    rs = np.where(q % 2 == 1, c0, s0) * np.where(q % 4 >= 2, -1, 1)
    rc = np.where(q % 2 == 1, s0, c0) * np.where((q + 1) % 4 >= 2, -1, 1)
    assert _ulps(s, rs) <= 0.76 and _ulps(c, rc) <= 0.76


def test_special_arguments(lib):
    assert list(_call(lib, "log_64", np.array([1.0]))) == [0.0]
    assert list(_call(lib, "sqrt_64", np.array([0.0, -0.0]))) == [0.0, 0.0]
    got = _call(lib, "log2_64", np.array([0.0, np.inf, -1.0, np.nan, 5e-324]))
    assert got[0] == -np.inf and got[1] == np.inf and np.isnan(got[2]) and np.isnan(got[3]) and got[4] == -1074.0


def test_cancelling_sums_of_the_solve(lib):
    """rh.r of r = s - omega t from rh.s and rh.t, t so near s / omega that r is a
    thousandth of s: as near to the exact value for the rounded r as the rounding
    of r allows, one unit of sum |rh_i r_i| (the sums in one part lose some fifty
    times that)."""
    from fractions import Fraction as F
    rng = np.random.default_rng(5)
    n, omega = 2000, 0.7310585786300049
    s, rh = rng.standard_normal(n), rng.standard_normal(n)
    t = (s * (1 + 1e-3 * rng.standard_normal(n))) / omega
    p = lambda a: ctypes.c_void_p(a.ctypes.data)
    lib.t_new_rho.restype = ctypes.c_double
    got = lib.t_new_rho(p(s), p(t), p(rh), ctypes.c_double(omega), ctypes.c_long(n))
    r = [float(F(a) - F(omega) * F(b)) for a, b in zip(s, t)]  # rounded once
    rho, unit = sum(F(x) * F(y) for x, y in zip(r, rh)), F(2.0 ** -52) * sum(abs(F(x) * F(y)) for x, y in zip(r, rh))
    assert abs(F(got) - rho) <= unit
    one = float(np.dot(rh, s) - omega * np.dot(rh, t))
    print("in one part: %.0f units" % (abs(F(one) - rho) / unit))
