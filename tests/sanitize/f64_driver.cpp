// Errors of csrc/f64_math.h on the host, in ulp of the long double value: name,
// root mean square, largest.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>

#define __device__
#define __forceinline__ inline
using std::fma;
using std::fmin;
static inline uint64_t bits(double v) {
    uint64_t u;
    std::memcpy(&u, &v, 8);
    return u;
}
static inline double value(uint64_t u) {
    double v;
    std::memcpy(&v, &u, 8);
    return v;
}
static inline int __double2loint(double v) { return (int)(uint32_t)bits(v); }
static inline int __double2hiint(double v) { return (int)(bits(v) >> 32); }
static inline double __hiloint2double(int h, int l) { return value((uint64_t)(uint32_t)h << 32 | (uint32_t)l); }
static inline double estimate(double v) { return value(bits(v) & ~((1ull << 30) - 1)); }
static inline int exponent(double v) {
    int e;
    (void)std::frexp(v, &e);
    return e;
}
static inline double mantissa(double v) {
    int e;
    return std::frexp(v, &e);
}
#define __builtin_amdgcn_rcp(x) estimate(1.0 / (x))
#define __builtin_amdgcn_rsq(x) estimate(1.0 / std::sqrt(x))
#define __builtin_amdgcn_frexp_mant mantissa
#define __builtin_amdgcn_frexp_exp exponent

#include "f64_math_host.h"

using namespace mdgmi::f64;

struct Error {
    double sum = 0, most = 0;
    long n = 0;
    void add(double v, long double ref) {
        int e;
        (void)frexpl(ref, &e);
        const double d = (double)((v - ref) / ldexpl(1.0L, e - 53));
        sum += d * d;
        most = std::fmax(most, std::fabs(d));
        n++;
    }
    void print(const char* name) const { std::printf("%s %.6f %.6f\n", name, std::sqrt(sum / n), most); }
};

int main() {
    std::mt19937_64 g(1);
    Error lg, lu, sq, dv, sn, cs, ex, dev;
    for (int i = 0; i < 1000000; i++) {
        const uint32_t wa = (uint32_t)g(), wb = (uint32_t)g();
        const double u1 = (wa + 0.5) * 2.3283064365386963e-10, u2 = (wb + 0.5) * 2.3283064365386963e-10;
        const double x = 1.0 + (double)(g() >> 11) * 0x1p-41, t = (double)(g() >> 11) * 0x1p-44;
        lg.add(ln_pos(x), logl(x));
        const double l = ln_pos(u1);
        lu.add(l, logl(u1));
        const double r = sqrt_pos(-2.0 * l), a = 6.283185307179586 * u2;
        sq.add(r, sqrtl(-2.0L * l));
        dv.add(fast_div(x, u1), (long double)x / u1);
        double s, c;
        sincos_turn(a, ((wb >> 29) + 1) >> 1, s, c);
        sn.add(s, sinl(a));
        cs.add(c, cosl(a));
        ex.add(exp_neg(t, exp_scale_unit()), expl(-(long double)t));
        dev.add(r * c, sqrtl(-2.0L * logl(u1)) * cosl(a));
    }
    lg.print("log"), lu.print("log_u"), sq.print("sqrt"), dv.print("div"), sn.print("sin"), cs.print("cos");
    ex.print("exp"), dev.print("deviate");
    return 0;
}
