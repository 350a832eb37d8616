// fp64 elementary functions for the ranges that the kernels meet, in a fraction
// of the general library routines' instructions (no scaling, special values or
// large arguments).  Arguments are finite; each function states its range.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace mcx {

// 1 / x to an ulp of fp64, for x away from zero and the range's ends (two
// Newton steps on the hardware's estimate)
__device__ __forceinline__ double fast_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// n / d likewise: the quotient's remainder corrects it once more, which gives
// the rounded quotient (to the last bit unless the reciprocal's own last bit
// is off and the quotient lies next to a rounding boundary)
__device__ __forceinline__ double fast_div(double n, double d) {
    const double r = fast_rcp(d);
    const double q = n * r;
    return __builtin_fma(__builtin_fma(-d, q, n), r, q);
}

// the same with r = fast_rcp(d) at hand
__device__ __forceinline__ double div_by(double n, double d, double r) {
    const double q = n * r;
    return __builtin_fma(__builtin_fma(-d, q, n), r, q);
}

// n / d for a constant d whose rounded reciprocal is inv
__device__ __forceinline__ double div_const(double n, double d, double inv) {
    const double q = n * inv;
    return __builtin_fma(__builtin_fma(-d, q, n), inv, q);
}

// 1 / sqrt(x) to an ulp or two, x away from zero and the range's ends
__device__ __forceinline__ double fast_rsqrt(double x) {
    double r = __builtin_amdgcn_rsq(x);
    const double hx = 0.5 * x;
    r = __builtin_fma(r, __builtin_fma(-hx * r, r, 0.5), r);
    return __builtin_fma(r, __builtin_fma(-hx * r, r, 0.5), r);
}

// sqrt(x), corrected once as fast_div's quotient is
__device__ __forceinline__ double fast_sqrt(double x) {
    const double r = fast_rsqrt(x);
    const double g = x * r;
    return __builtin_fma(__builtin_fma(-g, g, x), 0.5 * r, g);
}

// x^(-1/3) to an ulp or two for x in [1e-30, 1e30]: an fp32 estimate z (a few
// 1e-6 off) and the series of (1 - e)^(-1/3) in e = 1 - x z^3 to e^2, whose next
// term is below 2^-56
__device__ __forceinline__ double rcp_cbrt(double x) {
    const double z = (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf((float)x) * (-1.0f / 3.0f));
    const double e = __builtin_fma(-(x * (z * z)), z, 1.0);
    return __builtin_fma(z * e, __builtin_fma(e, 2.0 / 9.0, 1.0 / 3.0), z);
}

// exp(-t) for 0 <= t, within an ulp: t = n ln 2 - r with |r| <= ln(2) / 2 (ln 2
// in two parts, the first with trailing zeros so that n times it is exact) and
// the Taylor series of exp(r) to r^13 (its remainder is below 2^-57)
__device__ __forceinline__ double exp_neg(double t) {
    t = fmin(t, 800.0);                         // underflows to zero from 746 on
    const double n = __builtin_rint(t * 1.4426950408889634);
    double r = __builtin_fma(n, 0x1.62e42fefap-1, -t);
    r = __builtin_fma(n, 0x1.cf79abc9e3b3ap-40, r);
    constexpr double c[14] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720,
                              1.0 / 5040, 1.0 / 40320, 1.0 / 362880, 1.0 / 3628800,
                              1.0 / 39916800, 1.0 / 479001600, 1.0 / 6227020800.0};
    double e = c[13];
#pragma unroll
    for (int k = 12; k >= 0; --k) e = __builtin_fma(e, r, c[k]);
    return __builtin_ldexp(e, -(int)n);
}

// sine and cosine of x in [0, 2 pi]: reduced by multiples n of pi / 2 (in two
// parts; the products are exact in the fused multiply-adds), then the Taylor
// series on |r| <= pi / 4 to r^17 and r^16 (remainders below 2^-54)
__device__ __forceinline__ void sincos_2pi(double x, double &s, double &c) {
    const double n = __builtin_rint(x * 0.63661977236758134);
    double r = __builtin_fma(n, -0x1.921fb54442d18p+0, x);
    r = __builtin_fma(n, -0x1.1a62633145c07p-54, r);
    const double w = r * r;
    double ps = 1.0 / 355687428096000.0;
    ps = __builtin_fma(ps, w, -1.0 / 1307674368000.0);
    ps = __builtin_fma(ps, w, 1.0 / 6227020800.0);
    ps = __builtin_fma(ps, w, -1.0 / 39916800.0);
    ps = __builtin_fma(ps, w, 1.0 / 362880.0);
    ps = __builtin_fma(ps, w, -1.0 / 5040.0);
    ps = __builtin_fma(ps, w, 1.0 / 120.0);
    ps = __builtin_fma(ps, w, -1.0 / 6.0);
    ps = __builtin_fma(r * w, ps, r);
    double pc = 1.0 / 20922789888000.0;
    pc = __builtin_fma(pc, w, -1.0 / 87178291200.0);
    pc = __builtin_fma(pc, w, 1.0 / 479001600.0);
    pc = __builtin_fma(pc, w, -1.0 / 3628800.0);
    pc = __builtin_fma(pc, w, 1.0 / 40320.0);
    pc = __builtin_fma(pc, w, -1.0 / 720.0);
    pc = __builtin_fma(pc, w, 1.0 / 24.0);
    pc = __builtin_fma(w * w, pc, __builtin_fma(w, -0.5, 1.0));
    const int q = (int)n;                        // 0 .. 4
    const double a = (q & 1) ? pc : ps, b = (q & 1) ? ps : pc;
    s = (q & 2) ? -a : a;
    c = ((q + 1) & 2) ? -b : b;
}

// -log(u) for a positive fp32 u: u = m 2^e with m in [sqrt(1/2), sqrt(2)) and
// log m = 2 atanh(s), s = (m - 1) / (m + 1), its series to s^21 (remainder
// below 2^-56 of it)
__device__ __forceinline__ double neg_log(float u) {
    float m = __builtin_amdgcn_frexp_mantf(u);
    int e = __builtin_amdgcn_frexp_expf(u);
    const bool low = m < 0.70710677f;
    m = low ? 2.0f * m : m;
    e = low ? e - 1 : e;
    const double f = (double)m - 1.0;
    const double s = fast_div(f, 2.0 + f);
    const double w = s * s;
    double p = 1.0 / 21;
    p = __builtin_fma(p, w, 1.0 / 19);
    p = __builtin_fma(p, w, 1.0 / 17);
    p = __builtin_fma(p, w, 1.0 / 15);
    p = __builtin_fma(p, w, 1.0 / 13);
    p = __builtin_fma(p, w, 1.0 / 11);
    p = __builtin_fma(p, w, 1.0 / 9);
    p = __builtin_fma(p, w, 1.0 / 7);
    p = __builtin_fma(p, w, 1.0 / 5);
    p = __builtin_fma(p, w, 1.0 / 3);
    const double s2 = s + s;
    const double lm = __builtin_fma(s2 * w, p, s2);
    const double k = (double)e;
    return -__builtin_fma(k, 0x1.62e42fefa39efp-1, __builtin_fma(k, 0x1.abc9e3b39803fp-56, lm));
}

}  // namespace mcx
