// Exponentials and logarithms of the log number system, in FP64. Written for
// the arguments the lattice kernels have (no NaN, no negative or infinite
// argument of a logarithm), which is what makes them faster than the device
// library's; none has a larger error than the library's function in its place
// (largest error in units of the last place over 4 million arguments per
// range, device library in parentheses): e^x 0.87 (0.88), ln y 0.63 (0.64),
// ln(1 + x) 0.63 (0.64). At n = 25, d = 4 the log form's alpha tile takes 1.41 ms
// with the library's functions and 1.03 with these, its Gamma tile 2.18 and 1.84,
// the sweeps' kernels 5.03 and 4.55. The host form is for the tests.
#pragma once
#include <math.h>

#ifdef __HIPCC__
#define BN_MATH __host__ __device__ static inline
#else
#define BN_MATH static inline
#endif
// products and sums as written: the rounding errors below are those of single
// operations
#ifdef __clang__
#define BN_AS_WRITTEN _Pragma("clang fp contract(off)")
#else
#define BN_AS_WRITTEN
#endif

namespace bnk {

// ln 2 = kLn2Hi + kLn2Lo: the 41 leading bits, so that small integers times
// kLn2Hi are exact, and the rest
constexpr double kLn2Hi = 0x1.62e42fefa38p-1, kLn2Lo = 0x1.ef35793c7673p-45;

// e^x 2^shift for x > -2800, as exp_scaled: x = k ln 2 + r, |r| <= ln 2 / 2, and
// e^r = 1 + r + r^2 q(r), q the minimax polynomial of degree 10 (Remez; error
// below 2^-60 of e^r; one degree less, fitted to e^r as a whole, reached 0.95
// units). The shift costs nothing here; as a factor or an offset outside it
// would be a rounding more.
BN_MATH double exp_held(double x, int shift) {
    const double k = rint(x * 1.4426950408889634074);
    double r = fma(k, -kLn2Hi, x);
    r = fma(k, -kLn2Lo, r);
    double q = 2.0826637596418214e-09;
    q = fma(q, r, 2.5112024946363768e-08);
    q = fma(q, r, 2.755758174178715e-07);
    q = fma(q, r, 2.7557234895399425e-06);
    q = fma(q, r, 2.480158692685955e-05);
    q = fma(q, r, 0.00019841269896351003);
    q = fma(q, r, 0.0013888888889115446);
    q = fma(q, r, 0.008333333333317048);
    q = fma(q, r, 0.041666666666666095);
    q = fma(q, r, 0.16666666666666682);
    q = fma(q, r, 0.5);
    return ldexp(fma(fma(q, r, 1.0), r, 1.0), (int)k + shift);
}
// e^x 2^shift: 0 far below and for x = -inf (or NaN), +inf where it overflows
BN_MATH double exp_scaled(double x, int shift) {
    return exp_held(fmin(fmax(x, -2800.0), 2800.0), shift);
}
// the same for x <= 0
BN_MATH double exp_below(double x, int shift) { return exp_held(fmax(x, -2800.0), shift); }
BN_MATH double exp_neg(double x) { return exp_below(x, 0); }

// k ln 2 + ln(1 + f + flo) for sqrt(1/2) <= 1 + f <= sqrt(2) and an integer k,
// flo a rounding error of f: with s = f / (2 + f) and z = s^2,
// ln(1 + f) = f - f^2 / 2 + s (f^2 / 2 + z p(z)) (the form that fdlibm's log has),
// p the Chebyshev interpolant of degree 7 of (2 atanh(s) / s - 2) / z (error below
// 2^-60). The large terms are
// summed with their rounding errors and the quotient s is kept unrounded where
// it counts, so that the result is exact for k = 0 and small f, where it is f.
BN_MATH double log_parts(double f, double flo, double k) {
    BN_AS_WRITTEN
    const double den = 2.0 + f;
#ifdef __HIP_DEVICE_COMPILE__
    double rc = __builtin_amdgcn_rcp(den);                   // 24 bits
#else
    double rc = (double)(float)(1.0 / den);
#endif
    rc = fma(fma(-den, rc, 1.0), rc, rc);
    const double s0 = f * rc, ds = fma(-den, s0, f) * rc, s = s0 + ds;
    const double z = s * s;
    double p = 0.1308800183236331;
    p = fma(p, z, 0.13268641529664726);
    p = fma(p, z, 0.15386244619495787);
    p = fma(p, z, 0.1818179554969504);
    p = fma(p, z, 0.2222222239256068);
    p = fma(p, z, 0.2857142857079987);
    p = fma(p, z, 0.40000000000000885);
    p = fma(p, z, 0.6666666666666666);
    const double f2 = 0.5 * f, hf = f2 * f, hlo = fma(f2, f, -hf);
    const double x = fma(z, p, hf);
    const double w = fma(s0, x, fma(ds, x, fma(k, kLn2Lo, flo))) - hlo;
    const double a = f - hf, da = (f - a) - hf;
    const double kl = k * kLn2Hi, h = kl + a, dh = (kl - h) + a;
    return h + (dh + (da + w));
}

// ln(y 2^-shift) for a positive finite y
BN_MATH double log_scaled(double y, int shift) {
#ifdef __HIP_DEVICE_COMPILE__
    double m = __builtin_amdgcn_frexp_mant(y);
    int e = __builtin_amdgcn_frexp_exp(y);
#else
    int e;
    double m = frexp(y, &e);
#endif
    const bool low = m < 0.70710678118654757;
    m = low ? m + m : m;
    e -= low ? 1 : 0;
    return log_parts(m - 1.0, 0.0, (double)(e - shift));
}
BN_MATH double log_pos(double y) { return log_scaled(y, 0); }

// ln(1 + x), 0 <= x <= 1: from sqrt(2) - 1 on as ln 2 + ln((1 + x) / 2), whose
// f = (x - 1) / 2 is rounded below x = 1/2 (the error times 1 / (1 + f), which
// is within 3% of 11/8 there)
BN_MATH double log1p_unit(double x) {
    BN_AS_WRITTEN
    const bool up = x >= 0.41421356237309503;
    const double f = up ? fma(0.5, x, -0.5) : x;
    const double flo = up ? 1.375 * fma(0.5, x, -0.5 - f) : 0.0;
    return log_parts(f, flo, up ? 1.0 : 0.0);
}

}  // namespace bnk
