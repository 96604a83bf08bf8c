"""Accuracy of the Box-Muller pieces (csrc/bm_math.h), compiled for the host:
the cosine against an 80-bit reference, no further off than the two Taylor
series on [0, pi/4] evaluated plainly here; quotients and square roots equal
to the IEEE operations although the host starts them from 23 bits; values
taken four at a time equal to single ones; weights through these forms equal
to the library-function formula."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(HERE, "..", "paper_2512_09502_amd", "csrc", "bm_math.h")

SRC = r'''
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>
#include "HEADER"
using namespace snnc;
static bool same(double a, double b) { return std::memcmp(&a, &b, 8) == 0; }
// sine and cosine of 2 pi w / 2^32 from their series on [0, pi/4], and the first-order term of the double product
static double plain(uint32_t w) {
    const uint32_t q = w >> 30, r = w & 0x3fffffffu;
    const bool low = r < (1u << 29);
    const double b = (double)(low ? r : (1u << 30) - r) * 1.4629180792671596e-09, z = b * b;
    double s = 0, c = 0, f = 1;
    std::vector<double> fact(20, 1.0);
    for (int k = 1; k < 20; ++k) fact[k] = f *= k;
    for (int k = 19; k >= 3; k -= 2) s = s * z + ((k / 2) % 2 ? -1.0 : 1.0) / fact[k];
    for (int k = 18; k >= 2; k -= 2) c = c * z + ((k / 2) % 2 ? 1.0 : -1.0) / fact[k];
    const double sb = b + b * (z * s), cb = 1.0 - z * c, ca = low ? cb : sb, sa = low ? sb : cb;
    const double ct[4] = {ca, -sa, -ca, sa}, st[4] = {sa, ca, -sa, -ca};
    const double u = (double)w * (1.0 / 4294967296.0), x = 6.283185307179586 * u;
    return ct[q] - st[q] * (-2.4492935982947064e-16 * u - std::fma(6.283185307179586, u, -x));
}
int main() {
    std::mt19937_64 rng(11);
    double worst = 0, worst_plain = 0;
    long groups = 0, quot = 0, root = 0, weights = 0;
    for (long i = 0; i < 500000; ++i) {
        uint32_t w[4];
        uint64_t v[4];
        double c4[4], l4[4];
        for (int k = 0; k < 4; ++k) {
            w[k] = i < 200 ? (uint32_t)(((uint64_t)(i / 25) << 29) + (uint32_t)((int)(i % 25) * 4 + k - 50)) : (uint32_t)rng();
            v[k] = (uint64_t)w[k] + 1;
        }
        cos_2pi_u32s<4>(w, c4);
        log_u32_fracs<4>(v, l4);
        double x4[4], r4[4], n4[4], d4[4], q4[4];
        for (int k = 0; k < 4; ++k) {
            groups += !same(c4[k], cos_2pi_u32(w[k])) + !same(l4[k], log_u32_frac(v[k]));
            const long double ref = cosl((long double)(6.283185307179586 * ((double)w[k] * (1.0 / 4294967296.0))));
            worst = std::fmax(worst, (double)fabsl((long double)c4[k] - ref));
            worst_plain = std::fmax(worst_plain, (double)fabsl((long double)plain(w[k]) - ref));
            x4[k] = -2.0 * l4[k];
            const double m = 0.70710678 + 0.70710678 * ((double)v[k] * (1.0 / 4294967296.0));
            n4[k] = m - 1.0;
            d4[k] = m + 1.0;
        }
        square_roots<4>(x4, r4);
        quotients<4>(n4, d4, q4);
        for (int k = 0; k < 4; ++k) {
            root += r4[k] != std::sqrt(x4[k]);
            quot += q4[k] != n4[k] / d4[k];
            const double g[1] = {x4[k]};
            double y[1];
            square_roots<1>(g, y);
            groups += !same(y[0], r4[k]);
            const uint32_t w1 = w[(k + 1) & 3];
            volatile double zl = r4[k] * c4[(k + 1) & 3], sl = 0.05 * zl;
            volatile double rr = std::sqrt(-2.0 * std::log((double)v[k] * (1.0 / 4294967296.0)));
            volatile double zr = rr * std::cos(6.283185307179586 * ((double)w1 * (1.0 / 4294967296.0))), sr = 0.05 * zr;
            weights += (float)(-0.5 + sl) != (float)(-0.5 + sr);
        }
    }
    const double zero[1] = {0.0};
    double y[1];
    square_roots<1>(zero, y);
    std::printf("%.4e %.4e %ld %ld %ld %ld %g\n", worst, worst_plain, groups, quot, root, weights, y[0]);
}
'''


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_accuracy_of_the_box_muller_pieces():
    with tempfile.TemporaryDirectory() as d:
        src = os.path.join(d, "t.cpp")
        open(src, "w").write(SRC.replace("HEADER", os.path.abspath(HEADER)))
        exe = os.path.join(d, "t")
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-o", exe, src, "-lm"])
        out = subprocess.check_output([exe], timeout=120).decode().split()
    worst, worst_plain = float(out[0]), float(out[1])
    groups, quotients, roots, weights = (int(x) for x in out[2:6])
    print(f"largest error of the cosine {worst:.3e}, of the plain series {worst_plain:.3e}")
    assert worst <= worst_plain
    assert groups == 0 and quotients == 0 and roots == 0 and weights == 0
    assert float(out[6]) == 0.0
