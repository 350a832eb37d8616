// Host build of csrc/fp64_math.hpp against libm.  The device's reciprocal,
// reciprocal-square-root, exp2 and log2 estimates are stood in for by values
// off by more than the hardware's are.  Prints, one per line: fp32 mismatches of
// sine, cosine and -log over every uniform the transport can draw, then the
// largest relative errors of rcp_cbrt, exp_neg, fast_rcp, fast_rsqrt, fast_div.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#define __device__
#define __forceinline__ inline
static double cut(double r) {
    uint64_t b;
    std::memcpy(&b, &r, 8);
    b &= ~((1ull << 31) - 1);
    std::memcpy(&r, &b, 8);
    return r;
}
static double host_rcp(double x) { return cut(1.0 / x); }
static double host_rsq(double x) { return cut(1.0 / std::sqrt(x)); }
static float host_exp2(float x) { return std::exp2(x) * (1.0f + 2.4e-7f); }
static float host_log2(float x) { return std::log2(x) * (1.0f + 2.4e-7f); }
static float host_mant(float u) { int e; return std::frexp(u, &e); }
static int host_exp(float u) { int e; std::frexp(u, &e); return e; }
#define __builtin_amdgcn_rcp host_rcp
#define __builtin_amdgcn_rsq host_rsq
#define __builtin_amdgcn_exp2f host_exp2
#define __builtin_amdgcn_logf host_log2
#define __builtin_amdgcn_frexp_mantf host_mant
#define __builtin_amdgcn_frexp_expf host_exp
using std::fmin;
#include FP64_MATH_HEADER

int main() {
    using namespace mcx;
    long bad[3] = {0, 0, 0};
    for (uint32_t x = 0; x < (1u << 23); ++x) {
        const float u = (float)(2u * x + 1u) * 5.9604644775390625e-8f;
        const double a = 6.283185307179586 * (double)u;
        double s, c;
        sincos_2pi(a, s, c);
        bad[0] += (float)s != (float)std::sin(a);
        bad[1] += (float)c != (float)std::cos(a);
        bad[2] += (float)neg_log(u) != (float)-std::log((double)u);
    }
    double err[5] = {0, 0, 0, 0, 0};
    auto worst = [](double &e, long double got, long double ref) {
        e = std::fmax(e, (double)std::fabs(got / ref - 1.0L));
    };
    for (int i = 1; i <= 1000000; ++i) {
        const double y = std::pow(10.0, -12.0 * i / 1e6), t = 700e-6 * i;
        worst(err[0], rcp_cbrt(y), 1.0L / cbrtl((long double)y));
        worst(err[1], exp_neg(t), expl(-(long double)t));
        worst(err[2], fast_rcp(1.0 + t), 1.0L / (1.0L + t));
        worst(err[3], fast_rsqrt(1e-3 + t), 1.0L / sqrtl((long double)(1e-3 + t)));
        worst(err[4], fast_div(y, 1.0 + t), (long double)y / (1.0L + t));
    }
    for (long b : bad) std::printf("%ld\n", b);
    for (double e : err) std::printf("%.3e\n", e);
}
