// math64.hpp - float64 reciprocal, square root, logarithm and arctangent of the sweeps, for gfx950.
//
// The pairs of the float64 path spend most of their time in these.  Written for them instead of the
// library's functions: no branches, one reciprocal each, and the logarithm of a ratio from the difference
// of its terms.  Coefficients from csrc/fit_math64.py.  Errors against long double over 4e6 random
// arguments each (units of the last place): reciprocal 1.0, reciprocal square root 1.0, logarithm 1.1,
// logarithm of a ratio 1.9 (of the ratio's own rounding, which the difference avoids), arctangent 1.6.
#pragma once

#include <hip/hip_runtime.h>

namespace bem {

// 1 / d for normal d: the hardware's estimate (relative error e below 2^-22) times 1 + e + e^2 + e^3.
__device__ inline double rcp_f64(double d)
{
    const double r = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, r, 1.0);
    return fma(r, fma(e, fma(e, e, e), e), r);
}

// n / d for normal d, the quotient corrected by its remainder.
__device__ inline double div_f64(double n, double d)
{
    const double r = rcp_f64(d), q = n * r;
    return fma(fma(-d, q, n), r, q);
}

// 1 / sqrt(x) for normal x > 0: (1 - e)^(-1/2) to third order about the hardware's estimate.
__device__ inline double rsqrt_f64(double x)
{
    const double r = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * r, r, 1.0);
    return fma(r * e, fma(e, fma(e, 0.3125, 0.375), 0.5), r);
}

// P(z): atanh(s) = s (1 + z P(z)), z = s^2, |s| <= (sqrt 2 - 1) / (sqrt 2 + 1)
__device__ inline double atanh_poly(double z)
{
    double p = 0.06543426305539822;
    p = fma(p, z, 0.06634379044310099);
    p = fma(p, z, 0.07693119986394314);
    p = fma(p, z, 0.09090897820785153);
    p = fma(p, z, 0.1111111119581413);
    p = fma(p, z, 0.1428571428540219);
    p = fma(p, z, 0.20000000000000437);
    return fma(p, z, 0.3333333333333333);
}
// ln 2 = kLn2Hi + kLn2Lo, the head of 32 bits, so that its multiples by an exponent are exact
constexpr double kLn2Hi = 0.6931471803691238, kLn2Lo = 1.9082149292705877e-10;

// log x, x > 0: x = 2^e (1 + f), s = f / (2 + f), log(1 + f) = 2 atanh(s) = f - s (f - 2 z P(z))
__device__ inline double log_f64(double x)
{
    double m = __builtin_amdgcn_frexp_mant(x);       // [1/2, 1)
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.7071067811865476;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double f = m - 1.0, s = div_f64(f, 2.0 + f), z = s * s;
    const double r = 2.0 * z * atanh_poly(z);
    return fma((double)e, kLn2Hi, f - fma(s, f - r, -(double)e * kLn2Lo));
}

// log(b / a), a, b > 0, with the difference d = b - a given: for a ratio in [1 / sqrt 2, sqrt 2] it is
// 2 atanh(d / (a + b)), which keeps the relative accuracy of a small difference.
__device__ inline double log_ratio_f64(double a, double b, double d)
{
    const double ma = __builtin_amdgcn_frexp_mant(a), mb = __builtin_amdgcn_frexp_mant(b);
    int e = __builtin_amdgcn_frexp_exp(b) - __builtin_amdgcn_frexp_exp(a);
    e = mb > 1.4142135623730951 * ma ? e + 1 : e;
    e = mb < 0.7071067811865476 * ma ? e - 1 : e;
    const double bs = __builtin_amdgcn_ldexp(b, -e);
    const double num = e == 0 ? d : bs - a;
    const double s = div_f64(num, a + bs), z = s * s, t = s + s;
    return fma((double)e, kLn2Hi, t + fma((double)e, kLn2Lo, t * (z * atanh_poly(z))));
}

// atan(t) = t + t z p(z), z = t^2, |t| <= tan(pi / 16)
__device__ inline double atan_poly(double z)
{
    double p = -0.044903172480189366;
    p = fma(p, z, 0.05826811643531537);
    p = fma(p, z, -0.06664480286107828);
    p = fma(p, z, 0.07692257215801579);
    p = fma(p, z, -0.09090908404102156);
    p = fma(p, z, 0.11111111105850788);
    p = fma(p, z, -0.14285714285694098);
    p = fma(p, z, 0.1999999999999997);
    return fma(p, z, -0.3333333333333333);
}

// atan2(y, x): the octant's ratio n / d in [0, 1] is turned by 0, pi/8 or pi/4 (the nearest), as a
// quotient of the turned terms, and the remaining angle (at most pi/16) by a polynomial.  Where every lane's angle
// is small already (a segment or element five of its lengths away from all samples of the wavefront: most pairs) the
// turns and quadrants are left out, with the same result: 24 instructions instead of 55.
// Terms that are not normal numbers: beside an infinite one (samples beyond 1e154; x - 0.80 x bounds no small angle for it)
// the other is nothing; of two denormal ones (samples within 1e-306 of an element's end) the remaining angle is left out.
// (Scaling those instead, by selects or in a branch of its own, took 2 to 4% of the float64 adjoint.)
__device__ inline double atan2_f64(double y, double x)
{
    const double ax = fabs(x), ay = fabs(y);
    if (__all(ay < fma(-0.801087632620342, x, x))) {
        const double t = div_f64(y, x), z = t * t;
        return t + fma(t * z, atan_poly(z), 0.0);
    }
    const double d = fmax(ax, ay), n = fmin(ax, ay);
    const bool m1 = n > 0.198912367379658 * d, m2 = n > 0.6681786379192989 * d;
    const double c = m2 ? 1.0 : (m1 ? 0.41421356237309503 : 0.0);
    const double base = m2 ? 0.7853981633974483 : (m1 ? 0.39269908169872414 : 0.0);
    const double low = m2 ? 3.061616997868383e-17 : (m1 ? 3.060132146563891e-18 : 0.0);      // atan(c) - base
    const double num = fma(-c, d, n), den = fma(c, n, d);
    const double t = (d >= 0x1p-1022) & (d < INFINITY) ? div_f64(num, den) : 0.0;
    const double z = t * t;
    double r = base + (t + fma(t * z, atan_poly(z), low));
    r = ay > ax ? 1.5707963267948966 - (r - 6.123233995736766e-17) : r;
    r = x < 0.0 ? 3.141592653589793 - (r - 1.2246467991473532e-16) : r;
    r = __builtin_isunordered(x, y) ? x + y : r;
    return copysign(r, y);
}

}  // namespace bem
