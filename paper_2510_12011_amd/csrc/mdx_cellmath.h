// FP64 elementary functions of the cell models, for arguments a cell model
// forms.  Against the library's functions they issue fewer instructions at the
// same accuracy (about one unit in the last place): exp 17 against 42, log 35
// against 98, quotient 7 against 12.  Most of the difference is that the
// polynomials' coefficients sit in scalar registers (Coef, made once per
// thread), so each Horner step is one three-address FMA; as literals they cost
// a move into vector registers per step.  Against 80-bit arithmetic, over
// 60,000 cells with V and states drawn over their ranges, the current's rms error is
// 2.5e-16 of its rms with either (ten Tusscher-Panfilov), 2.5e-16 with the
// library's and 2.4e-16 with these (Courtemanche-Ramirez-Nattel).
//
// Polynomials: interpolation at Chebyshev nodes, computed in extended
// precision from the functions' power series.
//   expm1(r) = r + r^2 Q(r), |r| <= ln2 / 2: 4.1e-17 relative, 1.6e-17 of e^r
//   log((1 + f) / (1 - f)) = 2f + f^3 R(f^2), |f| <= (sqrt2 - 1) / (sqrt2 + 1):
//   5e-18 relative
#pragma once
#include <hip/hip_runtime.h>

namespace mdx {
namespace cell {

struct Coef {
    double q[10], r[7];
    double log2e, ln2hi, ln2lo;
};

__device__ __forceinline__ double scalar_const(double c)
{
    asm("" : "+s"(c));
    return c;
}

__device__ __forceinline__ Coef make_coef()
{
    return {{scalar_const(0x1.0000000000001p-1), scalar_const(0x1.5555555555556p-3),
             scalar_const(0x1.5555555553d55p-5), scalar_const(0x1.1111111110974p-7),
             scalar_const(0x1.6c16c17891317p-10), scalar_const(0x1.a01a01a7e02cap-13),
             scalar_const(0x1.a019b8f8d1f0dp-16), scalar_const(0x1.71de0d6518498p-19),
             scalar_const(0x1.28919d4d6a6e8p-22), scalar_const(0x1.af392a7cc96bfp-26)},
            {scalar_const(0x1.5555555555558p-1), scalar_const(0x1.9999999995274p-2),
             scalar_const(0x1.2492492dfd834p-2), scalar_const(0x1.c71c62d5e2662p-3),
             scalar_const(0x1.7462b91de4e47p-3), scalar_const(0x1.39fdcc7a88a4cp-3),
             scalar_const(0x1.2b5f6f43dddfbp-3)},
            scalar_const(0x1.71547652b82fep+0), scalar_const(-0x1.62e42fee00000p-1),
            scalar_const(-0x1.a39ef35793c76p-33)};
}

// Q of the reduced argument r = x - k ln2
__device__ __forceinline__ double exp_q(const Coef &c, double x, double &r, double &k)
{
    k = __builtin_rint(x * c.log2e);
    r = __builtin_fma(k, c.ln2hi, x);
    r = __builtin_fma(k, c.ln2lo, r);
    double q = c.q[9];
#pragma unroll
    for (int i = 8; i >= 0; --i) q = __builtin_fma(q, r, c.q[i]);
    return q;
}

// e^x for |x| < 1e10 (0 and infinity where it leaves the range)
__device__ __forceinline__ double exp_(const Coef &c, double x)
{
    double r, k;
    const double q = exp_q(c, x, r, k);
    const double p = __builtin_fma(__builtin_fma(q, r, 1.0), r, 1.0);
    return __builtin_amdgcn_ldexp(p, (int)k);
}

// e^x for x <= 0, any size
__device__ __forceinline__ double exp_neg(const Coef &c, double x)
{
    asm("v_max_f64 %0, %1, %2" : "=v"(x) : "v"(x), "s"(-800.0));
    return exp_(c, x);
}

// e^x and e^x - 1 for |x| <= 700
__device__ __forceinline__ void exp_expm1(const Coef &c, double x, double &e, double &em1)
{
    double r, k;
    const double q = exp_q(c, x, r, k);
    const double m = __builtin_fma(q * r, r, r);   // e^r - 1
    const double s = __builtin_amdgcn_ldexp(1.0, (int)k);
    em1 = __builtin_fma(s, m, s - 1.0);
    e = __builtin_fma(s, m, s);
}

// 1/x for x whose reciprocal is a normal number: the instruction's 24 bits and
// one third-order step (half a unit; 1/x and 1/y from one reciprocal of x y
// would save two instructions and lose a bit)
__device__ __forceinline__ double rcp(double x)
{
    const double y = __builtin_amdgcn_rcp(x), e = __builtin_fma(-x, y, 1.0);
    return __builtin_fma(y, __builtin_fma(e, e, e), y);
}

// x / y to half a unit and little more, for finite x / y and y as rcp() takes it
// (where a division gives 0 or infinity this gives NaN)
__device__ __forceinline__ double div(double x, double y)
{
    const double r = rcp(y), q = x * r;
    return __builtin_fma(__builtin_fma(-y, q, x), r, q);
}

// log(c) - log(x), log(c) given as hi + lo
__device__ __forceinline__ double log_ratio(const Coef &c, double hi, double lo, double x)
{
    // x = 2^e m, m in [sqrt(1/2), sqrt(2)): the exponent of x sqrt(1/2)
    const int e = __builtin_amdgcn_frexp_exp(x * 0.70710678118654752);
    const double m = __builtin_amdgcn_ldexp(x, -e);
    const double f = div(m - 1.0, m + 1.0), s = f * f;
    double q = c.r[6];
#pragma unroll
    for (int i = 5; i >= 0; --i) q = __builtin_fma(q, s, c.r[i]);
    const double ed = (double)e;
    double y = __builtin_fma(ed, c.ln2lo, lo) - f * s * q;
    y = __builtin_fma(-2.0, f, y);
    y = __builtin_fma(ed, c.ln2hi, hi) + y;
    // all but positive normal numbers (class bit 8)
    if (__builtin_expect(!__builtin_amdgcn_class(x, 0x100), 0)) y = hi - log(x);
    return y;
}

// x (hi + lo), lo what the rounding of a constant to hi leaves
__device__ __forceinline__ double times(double x, double hi, double lo)
{
    return __builtin_fma(x, hi, x * lo);
}

// x held in [-lim, lim]; NaN stays
__device__ __forceinline__ double clip(double x, double lim)
{
    x = x < -lim ? -lim : x;
    return x > lim ? lim : x;
}

}  // namespace cell
}  // namespace mdx
