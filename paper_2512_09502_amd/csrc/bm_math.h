// Double-precision pieces of the Box-Muller normal for 32-bit uniform words,
// written for the arguments that occur there (usable on host and device):
// ln(v / 2^32) for integer v in [1, 2^32] and cos(2 pi w / 2^32) for a word w.
// Both reduce their argument exactly with integer operations, so only short
// polynomials remain (Taylor series of atanh, sin and cos, truncated below
// 2^-56 on the reduced ranges).
#pragma once

#include <cmath>
#include <cstdint>
#include <cstring>

#ifndef __HIPCC__
#define SNNC_HD inline
#define SNNC_UNROLL
#else
#define SNNC_HD __host__ __device__ __forceinline__
#define SNNC_UNROLL _Pragma("unroll")
#endif

namespace snnc {

#ifdef __HIP_DEVICE_COMPILE__
// hardware reciprocal and reciprocal square root (about 1e-8 relative), to be refined
SNNC_HD double approx_rcp(double x) { return __builtin_amdgcn_rcp(x); }
SNNC_HD double approx_rsq(double x) { return __builtin_amdgcn_rsq(x); }
#else
// 23 significant bits, fewer than the hardware's: a host check then sees the refinement work
SNNC_HD double leading_bits(double x) {
    uint64_t u;
    std::memcpy(&u, &x, 8);
    u &= ~0ull << 30;
    std::memcpy(&x, &u, 8);
    return x;
}
SNNC_HD double approx_rcp(double x) { return leading_bits(1.0 / x); }
SNNC_HD double approx_rsq(double x) { return leading_bits(1.0 / std::sqrt(x)); }
#endif

// The functions take N arguments in lockstep: a coefficient is then brought
// into registers once for N steps of Horner's rule.  One value at a time, half
// as many moves as multiply-adds were issued for the coefficients.

// n / d for 1 <= d <= 4: the reciprocal refined by two Newton steps, the
// quotient by its remainder (Markstein, IBM J. Res. Dev. 34, 1990; no scaling:
// neither end of the exponent range occurs).  On the device equal to n / d for
// each of the 2^32 arguments of the logarithm below.
template <int N>
SNNC_HD void quotients(const double (&n)[N], const double (&d)[N], double (&q)[N]) {
    double r[N];
    SNNC_UNROLL for (int i = 0; i < N; ++i) r[i] = approx_rcp(d[i]);
    SNNC_UNROLL for (int i = 0; i < N; ++i) r[i] = fma(r[i], fma(-d[i], r[i], 1.0), r[i]);
    SNNC_UNROLL for (int i = 0; i < N; ++i) r[i] = fma(r[i], fma(-d[i], r[i], 1.0), r[i]);
    SNNC_UNROLL for (int i = 0; i < N; ++i) q[i] = n[i] * r[i];
    SNNC_UNROLL for (int i = 0; i < N; ++i) q[i] = fma(fma(-d[i], q[i], n[i]), r[i], q[i]);
}

// square roots of x in [0, 64]: y = x rsq(x) refined by a Newton step on y and
// on 1 / (2 y) together (Goldschmidt's iteration; Markstein, RNC 6, 2004), then
// twice by y's remainder.  On the device equal to sqrt(x) for each of the 2^32
// values of -2 ln(v / 2^32).
template <int N>
SNNC_HD void square_roots(const double (&x)[N], double (&y)[N]) {
    double g[N], h[N];
    SNNC_UNROLL for (int i = 0; i < N; ++i) {
        const double r = approx_rsq(x[i]);
        g[i] = x[i] * r;
        h[i] = 0.5 * r;
    }
    SNNC_UNROLL for (int i = 0; i < N; ++i) {
        const double e = fma(-h[i], g[i], 0.5);
        g[i] = fma(g[i], e, g[i]);
        h[i] = fma(h[i], e, h[i]);
    }
    SNNC_UNROLL for (int i = 0; i < N; ++i) g[i] = fma(fma(-g[i], g[i], x[i]), h[i], g[i]);
    SNNC_UNROLL for (int i = 0; i < N; ++i) g[i] = fma(fma(-g[i], g[i], x[i]), h[i], g[i]);
    SNNC_UNROLL for (int i = 0; i < N; ++i) y[i] = x[i] > 0.0 ? g[i] : 0.0;
}

// ln(v / 2^32), v in [1, 2^32].  v = m 2^e with m in [sqrt(1/2), sqrt(2)),
// ln m = 2 atanh(s), s = (m - 1) / (m + 1), |s| <= 0.1716; ln 2 in two parts
// so that e ln2_hi is exact.
template <int N>
SNNC_HD void log_u32_fracs(const uint64_t (&v)[N], double (&out)[N]) {
    const double ln2_hi = 0.6931471803691238;      // ln 2 with 32 significant bits
    const double ln2_lo = 1.9082149292705877e-10;  // ln 2 - ln2_hi
    // 1 / (2k + 1), k = 11 .. 1: atanh(s) / s = sum z^k / (2k + 1), k = 0 .. 11
    const double c[11] = {1.0 / 23.0, 1.0 / 21.0, 1.0 / 19.0, 1.0 / 17.0, 1.0 / 15.0, 1.0 / 13.0,
                          1.0 / 11.0, 1.0 / 9.0,  1.0 / 7.0,  1.0 / 5.0,  1.0 / 3.0};
    int e[N];
    double num[N], den[N], s[N], z[N], p[N];
    SNNC_UNROLL for (int i = 0; i < N; ++i) {
        e[i] = 63 - __builtin_clzll(v[i]);               // v >= 1
        double m = ldexp((double)v[i], -e[i]);           // exact
        if (m > 1.4142135623730951) {
            m *= 0.5;
            e[i] += 1;
        }
        num[i] = m - 1.0;
        den[i] = m + 1.0;
    }
    quotients<N>(num, den, s);
    SNNC_UNROLL for (int i = 0; i < N; ++i) {
        z[i] = s[i] * s[i];
        p[i] = c[0];
    }
    SNNC_UNROLL for (int k = 1; k < 11; ++k)
        SNNC_UNROLL for (int i = 0; i < N; ++i) p[i] = p[i] * z[i] + c[k];
    SNNC_UNROLL for (int i = 0; i < N; ++i) {
        const double ln_m = 2.0 * s[i] + 2.0 * s[i] * (z[i] * p[i]);
        const double k = (double)(e[i] - 32);
        out[i] = k * ln2_hi + (k * ln2_lo + ln_m);
    }
}

// cos(x) for x = fl(2pi_d * w / 2^32), the argument as a double product
// (2pi_d = 2 pi rounded to double), as Box-Muller in double precision forms
// it.  theta = 2 pi w / 2^32 is reduced exactly: quadrant q = w >> 30, the
// offset r inside it folded to [0, pi/4] (cos a = sin(pi/2 - a)), sine and
// cosine there by their Taylor series; then x = theta + corr with
// corr = (2pi_d - 2 pi) u + (the product's rounding error, exact by a fused
// multiply-add), so cos x = cos theta - corr sin theta (corr <= 1e-15: the
// next term is below 1e-30).  One sine series on [0, pi/2] saves nine
// multiply-adds, but its largest error is 2.5e-16 instead of 2.2e-16.
template <int N>
SNNC_HD void cos_2pi_u32s(const uint32_t (&w)[N], double (&out)[N]) {
    const double two_pi_over_2_32 = 1.4629180792671596e-09;   // 2 pi / 2^32
    const double two_pi_d = 6.283185307179586;                 // 2 pi rounded to double
    const double two_pi_err = -2.4492935982947064e-16;         // two_pi_d - 2 pi
    // sin b = b - b^3/3! + b^5/5! - ... (to b^19), cos b = 1 - b^2/2! + b^4/4! - ... (to b^18), b^2 <= 0.617
    const double cs[9] = {-1.0 / 121645100408832000.0, 1.0 / 355687428096000.0, -1.0 / 1307674368000.0,
                          1.0 / 6227020800.0,          -1.0 / 39916800.0,       1.0 / 362880.0,
                          -1.0 / 5040.0,               1.0 / 120.0,             -1.0 / 6.0};
    const double cc[9] = {1.0 / 6402373705728000.0, -1.0 / 20922789888000.0, 1.0 / 87178291200.0,
                          -1.0 / 479001600.0,       1.0 / 3628800.0,         -1.0 / 40320.0,
                          1.0 / 720.0,              -1.0 / 24.0,             1.0 / 2.0};
    double b[N], z[N], q[N], p[N];
    SNNC_UNROLL for (int i = 0; i < N; ++i) {
        const uint32_t r = w[i] & 0x3fffffffu;
        b[i] = (double)(r < (1u << 29) ? r : (1u << 30) - r) * two_pi_over_2_32;
        z[i] = b[i] * b[i];
        q[i] = cs[0];
        p[i] = cc[0];
    }
    SNNC_UNROLL for (int k = 1; k < 9; ++k)
        SNNC_UNROLL for (int i = 0; i < N; ++i) {
            q[i] = q[i] * z[i] + cs[k];
            p[i] = p[i] * z[i] + cc[k];
        }
    SNNC_UNROLL for (int i = 0; i < N; ++i) {
        const double sb = b[i] + b[i] * (z[i] * q[i]), cb = 1.0 - z[i] * p[i];
        const bool cosine = (((w[i] >> 29) ^ (w[i] >> 30)) & 1u) == 0;   // the lower half of an even quadrant, the upper of an odd one
        const double c1 = cosine ? cb : sb, s1 = cosine ? sb : cb;
        const double ct = ((w[i] + (1u << 30)) >> 31) ? -c1 : c1;       // cos theta: negative in quadrants 1 and 2
        const double st = (w[i] >> 31) ? -s1 : s1;                      // sin theta: negative in quadrants 2 and 3
        const double u = (double)w[i] * (1.0 / 4294967296.0);
        const double x = two_pi_d * u;
        const double corr = two_pi_err * u - fma(two_pi_d, u, -x);      // x - 2 pi u
        out[i] = ct - st * corr;
    }
}

SNNC_HD double log_u32_frac(uint64_t v) {
    const uint64_t a[1] = {v};
    double out[1];
    log_u32_fracs<1>(a, out);
    return out[0];
}

SNNC_HD double cos_2pi_u32(uint32_t w) {
    const uint32_t a[1] = {w};
    double out[1];
    cos_2pi_u32s<1>(a, out);
    return out[0];
}

}  // namespace snnc
