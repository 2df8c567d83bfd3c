// FP64 exponential, division and logarithm of the FP64 kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace mdgmi {
namespace f64 {

// exp(-t) of t = d / (2 sigma2), d >= 0, as 2^-(d c) with c = log2(e) / (2 sigma2):
// the argument is rounded to an integer n by adding 1.5 2^52 (whose low word
// then holds n), the remainder f, |f| <= 1/2, is formed with c in two parts, so
// that d c itself is never rounded, and n goes into the exponent field of
// 2^f = 1 + f P(f), P the Chebyshev interpolant of degree 10 of (2^f - 1) / f
// (within 2e-17 of 2^f). d is capped where the result is 2^-1000 (this also
// takes NaN, to 2^-1000), so the field cannot wrap. About 1 ulp, 17
// instructions; a table of 2^(k/32) and a series of degree 6 take as many, and
// wait for the table.
struct ExpScale {
    double c, clo, dmax;
};

__device__ __forceinline__ ExpScale exp_scale(double inv2s2) {
    const double l = 0x1.71547652b82fep+0, ll = 0x1.777d0ffda0d24p-56;  // log2(e), two parts
    ExpScale e;
    const double c = inv2s2 * l;
    e.c = -c;
    e.clo = -fma(inv2s2, ll, fma(inv2s2, l, -c));
    e.dmax = 1000.0 / c;
    return e;
}

// exp(-d) itself
__device__ __forceinline__ ExpScale exp_scale_unit() {
    return {-0x1.71547652b82fep+0, -0x1.777d0ffda0d24p-56, 693.0};
}

constexpr double kExp2P[11] = {0x1.62e42fefa39efp-1,  0x1.ebfbdff82c598p-3,  0x1.c6b08d704a0c2p-5,
                               0x1.3b2ab6fba1ddap-7,  0x1.5d87fe78a5276p-10, 0x1.430913096fd9fp-13,
                               0x1.ffcbfc670dcd4p-17, 0x1.62bfd47773353p-20, 0x1.b524fae627834p-24,
                               0x1.e6063f7217bc6p-28, 0x1.e9d3fe3952179p-32};

__device__ __forceinline__ double exp_neg(double d, const ExpScale& s) {
    const double magic = 6755399441055744.0;  // 1.5 2^52
    d = fmin(d, s.dmax);
    const double b = fma(d, s.c, magic);
    const int n = __double2loint(b);
    const double r = b - magic;
    double f = fma(d, s.c, -r);
    f = fma(d, s.clo, f);
    double p = kExp2P[10];
#pragma unroll
    for (int k = 9; k >= 0; k--) p = fma(p, f, kExp2P[k]);
    const double v = fma(f, p, 1.0);
    return __hiloint2double(__double2hiint(v) + (n << 20), __double2loint(v));
}

// a / b for normal a, b and quotient (no range scaling): v_rcp_f64, a Newton step
// (45 bits from its 22 or more) and Markstein's residual correction, which makes
// up for the rest: within 0.5 ulp but for rare last bits.
__device__ __forceinline__ double fast_div(double a, double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(fma(-b, r, 1.0), r, r);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}

// ln x for normal positive x, within about 1 ulp: x = 2^e v, v in [sqrt(1/2),
// sqrt(2)), f = v - 1 (exact), s = f / (2 + f), and the atanh series ln v =
// 2 s + s R(s^2) with R its terms from 2/3 s^2 on, to s^20 (the next is below
// 3e-17), put together as f - s (f - R) so that s needs no extra digits (that
// regrouping, and ln 2 in two parts, as in fdlibm's logarithm). A third of the
// library log's instructions, whose two-word arithmetic has no use here: the sums
// it is taken of carry more than its rounding.
__device__ __forceinline__ double ln_pos(double x) {
    double v = __builtin_amdgcn_frexp_mant(x);  // [1/2, 1)
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = v < 0.70710678118654752440;
    v = low ? v + v : v;
    e -= low ? 1 : 0;
    const double f = v - 1.0, s = fast_div(f, 2.0 + f), z = s * s;
    double R = 2.0 / 21.0;
#pragma unroll
    for (int k = 19; k >= 3; k -= 2) R = fma(R, z, 2.0 / k);
    R *= z;
    const double de = (double)e;
    // ln 2 in two parts, the first with 21 trailing zero bits: de times it is exact
    return fma(de, 0x1.62e42fee00000p-1, f - fma(s, f - R, -de * 0x1.a39ef35793c76p-33));
}

// ln(1 + x) for x >= 0 up to the largest normal value
__device__ __forceinline__ double ln1p_pos(double x) {
    const double u = 1.0 + x;
    return ln_pos(u) + (x - (u - 1.0)) * __builtin_amdgcn_rcp(u);
}

// sqrt x for x and its root well inside the normal range (no range scaling):
// v_rsq_f64, one step of Goldschmidt's coupled iteration for root and half its
// reciprocal (45 bits from 22 or more), and Markstein's residual correction:
// within 0.5 ulp but for rare last bits.
__device__ __forceinline__ double sqrt_pos(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, x), h, g);
}

// sine and cosine of a in [0, 2 pi], k the multiple of pi / 2 next to it (0 to
// 4): a - k fl(pi / 2) is exact in one fma, a second one takes the rest of
// pi / 2 off, so the remainder r carries 53 bits also next to a zero. Chebyshev
// interpolants in z = r^2 up to (pi / 4)^2 of (sin r - r) / (r z) and
// (cos r - 1 + z / 2) / z^2, degree 5: 2e-17 and 1e-18 off (what 1 - z / 2 loses to
// rounding goes back in with the series, as in fdlibm's cosine, and so does what r
// itself loses, rl: 0.29 ulp root mean square and 0.8 at most (0.36 and 1.4 without
// rl; a correctly rounded result 0.289 and 0.5).
__device__ __forceinline__ void sincos_turn(double a, uint32_t k, double& sn, double& cs) {
    constexpr double S[6] = {-0x1.5555555555555p-3, 0x1.1111111110bb2p-7,   -0x1.a01a019e83aaep-13,
                             0x1.71de37968a024p-19, -0x1.ae600b02a7c74p-26, 0x1.5e0b19f38405ap-33};
    constexpr double C[6] = {0x1.5555555555555p-5,   -0x1.6c16c16c16967p-10, 0x1.a01a019f4eb00p-16,
                             -0x1.27e4fa17da030p-22, 0x1.1eeb68e934339p-29,  -0x1.907da36274fc5p-37};
    const double kd = (double)k;
    const double r0 = fma(-kd, 0x1.921fb54442d18p+0, a);
    const double r = fma(-kd, 0x1.1a62633145c07p-54, r0), rl = fma(-kd, 0x1.1a62633145c07p-54, r0 - r);
    const double z = r * r, w = fma(-0.5, z, 1.0);
    double s = S[5], c = C[5];
#pragma unroll
    for (int i = 4; i >= 0; i--) {
        s = fma(s, z, S[i]);
        c = fma(c, z, C[i]);
    }
    s = r + fma(r * z, s, rl * w);
    c = w + fma(z * z, c, fma(-r, rl, fma(-0.5, z, 1.0 - w)));
    const bool odd = k & 1;
    const double s1 = odd ? c : s, c1 = odd ? s : c;
    sn = __hiloint2double(__double2hiint(s1) ^ (int)((k << 30) & 0x80000000u), __double2loint(s1));
    cs = __hiloint2double(__double2hiint(c1) ^ (int)(((k + 1) << 30) & 0x80000000u), __double2loint(c1));
}

}  // namespace f64
}  // namespace mdgmi
