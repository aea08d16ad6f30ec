// gm_math.h -- FP64 elementary functions of the EM iterations and of the
// sampling, without the library's argument cases.  No HIP header is needed:
// with __device__ and __forceinline__ defined away and the four hardware
// estimates supplied, the same text compiles for the host, where the tests
// measure its error.
//
// The library's functions answer every argument; these have arguments of
// known range and can leave the cases out.  They are not to cost accuracy for
// it, so wherever a rounding would enter at full weight (a quotient, a leading
// product, the sum with the exponent) its error is carried along: what is left
// is the rounding of the last addition plus the roundings of terms that are a
// few percent of the result.  Largest error in units in the last place, on six
// million arguments each on the GPU (library's beside it): log2 0.57 (0.69),
// log 0.56 (0.64), sin and cos 0.71 (0.87), square root 0.50 (0.50), reciprocal
// 0.50 (0.50), reciprocal square root 0.99 (1.49 of root and quotient).
#pragma once

namespace gm {

// Reciprocal and reciprocal square root: two Newton steps on the hardware's
// estimates (about 2^-24) leave 0.5 and 1.0 units in the last place; 5 and 9
// instructions against 12 of the correctly rounded division and 27 of the
// square root and division.  For finite positive arguments.
__device__ __forceinline__ double rcp64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

__device__ __forceinline__ double rsq64(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// x = 2^e m with m in [sqrt(1/2), sqrt 2), and s = (m - 1) / (m + 1) as s + sl:
// m - 1 is exact, the rounding of m + 1 and the remainder of the quotient go
// into sl.  log m = 2 (s + s^3/3 + s^5/5 + ...) with |s| <= 0.172: the eleven
// terms kept leave 2e-18.
struct LogParts {
    double e, s, sl, z, q;  // z = s^2; q: the series from s^3 on over s^3
};
__device__ __forceinline__ LogParts log_parts(double x)
{
#pragma clang fp contract(off)
    LogParts p;
    double m = __builtin_amdgcn_frexp_mant(x);  // [1/2, 1)
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.70710678118654752440;
    m = low ? m + m : m;
    p.e = (double)(low ? e - 1 : e);
    const double n = m - 1.0, d = m + 1.0, dl = m - (d - 1.0), r = rcp64(d);
    p.s = n * r;
    p.sl = r * fma(-p.s, dl, fma(-p.s, d, n));
    p.z = p.s * p.s;
    double q = 1.0 / 21.0;
    q = fma(q, p.z, 1.0 / 19.0);
    q = fma(q, p.z, 1.0 / 17.0);
    q = fma(q, p.z, 1.0 / 15.0);
    q = fma(q, p.z, 1.0 / 13.0);
    q = fma(q, p.z, 1.0 / 11.0);
    q = fma(q, p.z, 1.0 / 9.0);
    q = fma(q, p.z, 1.0 / 7.0);
    q = fma(q, p.z, 1.0 / 5.0);
    p.q = fma(q, p.z, 1.0 / 3.0);
    return p;
}

// e + t + small with the rounding of e + t kept; e is 0 or above |t|
__device__ __forceinline__ double log_sum(double e, double t, double small)
{
#pragma clang fp contract(off)
    const double h = e + t;
    return h + ((t - (h - e)) + small);
}

// log2, 2 / ln 2 in two parts; of zero, infinities, negative values and NaN
// what the library gives (chosen at the end: a branch per value costs the
// iterations' builds registers)
__device__ __forceinline__ double log2_64(double x)
{
#pragma clang fp contract(off)
    const LogParts p = log_parts(x);
    const double c = 2.8853900817779268, cl = 4.0710547481862066e-17;
    const double t = c * p.s;
    const double tl = fma(c, p.s, -t) + fma(c, p.sl, cl * p.s);
    const double y = log_sum(p.e, t, fma(t * p.z, p.q, tl));
    const double special = x > 0.0 ? x : (x == 0.0 ? -__builtin_inf() : __builtin_nan(""));
    return x > 0.0 && x <= 1.7976931348623157e308 ? y : special;
}

// log of x in (0, 1]: ln 2 in two parts, the first with eleven trailing zero
// bits, so that its product with e is exact
__device__ __forceinline__ double log_64(double x)
{
#pragma clang fp contract(off)
    const LogParts p = log_parts(x);
    const double t = p.s + p.s;
    const double small = fma(t * p.z, p.q, fma(p.e, 5.497923018708371e-14, p.sl + p.sl));
    return log_sum(p.e * 0.6931471805598903, t, small);
}

// sqrt of x >= 0: rsq64 and one correction by the remainder
__device__ __forceinline__ double sqrt_64(double x)
{
    const double y = rsq64(x);
    const double g = x * y;
    return x > 0.0 ? fma(0.5 * y, fma(-g, g, x), g) : 0.0;
}

// sin and cos of pi a, a in [0, 2): a = q/2 + f exactly, |f| <= 1/4, and the
// Taylor series of both about 0 (nine terms leave 1e-19 and 2e-18), the
// leading products with their roundings, pi and pi^2 / 2 in two parts
__device__ __forceinline__ void sincospi_64(double a, double& sn, double& cs)
{
#pragma clang fp contract(off)
    const double h = __builtin_rint(a + a);
    const int q = (int)h;
    const double f = fma(-0.5, h, a);
    const double z = f * f, zl = fma(f, f, -z);
    double p = 7.95205400147551261113e-07;
    p = fma(p, z, -2.19153534478302172922e-05);
    p = fma(p, z, 4.66302805767612553716e-04);
    p = fma(p, z, -7.37043094571435044443e-03);
    p = fma(p, z, 8.21458866111282326461e-02);
    p = fma(p, z, -5.99264529320792105338e-01);
    p = fma(p, z, 2.55016403987734552317e+00);
    p = fma(p, z, -5.16771278004997025590e+00);
    const double x = f * 3.141592653589793;
    const double xl = fma(f, 3.141592653589793, -x) + f * 1.2246467991473532e-16;
    const double s0 = x + fma(f * z, p, xl);
    double c = 4.30306958703294729370e-06;
    c = fma(c, z, -1.04638104924845704697e-04);
    c = fma(c, z, 1.92957430940392314460e-03);
    c = fma(c, z, -2.58068913900140611828e-02);
    c = fma(c, z, 2.35330630358893205800e-01);
    c = fma(c, z, -1.33526276885458949906e+00);
    c = fma(c, z, 4.05871212641676848421e+00);
    const double w = -4.934802200544679 * z;
    const double wl = fma(-4.934802200544679, z, -w) + fma(-4.934802200544679, zl, -3.1326477543698557e-16 * z);
    const double g = 1.0 + w;
    const double c0 = g + ((w - (g - 1.0)) + fma(z * z, c, wl));
    const bool odd = (q & 1) != 0;
    const double u = odd ? c0 : s0, v = odd ? s0 : c0;
    sn = (q & 2) ? -u : u;
    cs = ((q + 1) & 2) ? -v : v;
}

// A sum carried as hi + lo (the exact error of every addition to hi goes to
// lo; Knuth's two-sum, and the product's error by fma): differences of such
// sums may cancel without losing what single ones would.
struct Sum2 {
    double hi, lo;
};
__device__ __forceinline__ void add2(Sum2& a, const Sum2& b)
{
#pragma clang fp contract(off)
    const double s = a.hi + b.hi, t = s - a.hi;
    a.lo += b.lo + ((a.hi - (s - t)) + (b.hi - t));
    a.hi = s;
}
// a += x y
__device__ __forceinline__ void mul_add2(Sum2& a, double x, double y)
{
#pragma clang fp contract(off)
    const double p = x * y;
    add2(a, Sum2{p, fma(x, y, -p)});
}
// a - w b
__device__ __forceinline__ Sum2 sub_scaled2(Sum2 a, double w, const Sum2& b)
{
#pragma clang fp contract(off)
    const double p = w * b.hi;
    add2(a, Sum2{-p, -fma(w, b.lo, fma(w, b.hi, -p))});
    return a;
}
__device__ __forceinline__ double value2(const Sum2& a) { return a.hi + a.lo; }

}  // namespace gm
