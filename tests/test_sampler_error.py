"""The rounding error of the plain sampler's FP64 arithmetic (cs_device.h) by
range of x, on the CPU: the header compiled for the host, with the hardware's
reciprocal, square-root, logarithm and exponential estimates replaced by
rounded ones of about their precision, against the same root and integral in
80-bit arithmetic.

Bounds: the rms error that the three-series / log1p form, which these replaced,
has on the same inputs (v by Halley's iteration on it from the table's total),
rounded up to three digits, for each range."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2206_02937_amd", "csrc")

SHIM = r"""
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
using std::fma; using std::isfinite;
#define __device__
#define __constant__
#define __forceinline__ inline
static inline double rounded(double r, int bits) {  // to that many bits
    if (!std::isfinite(r) || r == 0.0) return r;
    int e; const double m = std::frexp(r, &e);
    return std::ldexp(std::round(std::ldexp(m, bits)), e - bits);
}
static inline double rcp64(double a) { return rounded(1.0 / a, 26); }
static inline double rsq64(double a) { return rounded(1.0 / std::sqrt(a), 26); }
static inline float rcp32(float a) { return (float)(1.0 / (double)a); }
static inline float log32(float a) { return (float)std::log2((double)a); }
static inline float exp32(float a) { return (float)std::exp2((double)a); }
static inline float med3(float a, float b, float c) {
    return std::isnan(a) ? std::min(b, c) : std::max(std::min(a, b), std::min(std::max(a, b), c));
}
static inline double frexp_m(double a) { int e; return std::frexp(a, &e); }
static inline int frexp_e(double a) { int e; std::frexp(a, &e); return e; }
static inline int __clz(unsigned v) { return v ? __builtin_clz(v) : 32; }
static inline int __double2hiint(double x) { int64_t b; std::memcpy(&b, &x, 8); return (int)(b >> 32); }
static inline double __hiloint2double(int h, int l) {
    const int64_t b = ((int64_t)h << 32) | (uint32_t)l; double x; std::memcpy(&x, &b, 8); return x;
}
static inline void sincospi(double a, double* s, double* c) { *s = std::sin(M_PI * a); *c = std::cos(M_PI * a); }
"""

MAIN = r"""
typedef long double Q;
// T(v): one series below z = 1/2 or x = 1/2, the integrals as they stand above
static Q tail(Q v, Q x) {
    const Q z = x * v, A = 1 + z, first = v * (2 + z) / (2 * A * A);
    if (z < 0.5L || x < 0.5L) {
        const Q s = z / (2 + z), q = v / (2 + z), sg = s * s;
        Q p = 0, t = 1;
        for (int k = 0; k < 200 && t > 1e-22L; ++k, t *= sg) p += 2 * t / (2 * k + 3);
        return first + q * (2 - v * (2 - v) / A) + q * q * q * (x * x - 2 * x - 2) * p;
    }
    const Q l = log1pl(z), p2 = l - z / A, p3 = z - 2 * l + z / A;
    return first + l / x - (2 * p2 - p3 / x) / (x * x);
}
static Q root(Q target, Q x, Q v) {
    Q lo = 0, hi = 2;
    for (int i = 0; i < 200; ++i) {
        const Q R = tail(v, x) - target, a = 1 + x * v, f = 1 / (a * a * a) + 1 / a - v * (2 - v) / (a * a);
        (R > 0 ? hi : lo) = v;
        Q n = v - R / f;
        if (!(n > lo && n < hi)) n = (lo + hi) / 2;
        const Q d = n - v;
        v = n;
        if (fabsl(d) <= 1e-18L * v) break;
    }
    return v;
}
int main(int, char** arg) {
    const double x0 = atof(arg[1]), x1 = atof(arg[2]);
    const int n = atoi(arg[3]);
    std::mt19937_64 r(20260);
    std::uniform_real_distribution<double> U(0, 1);
    double sv = 0, ss = 0;
    for (int i = 0; i < n; ++i) {
        const double x = std::exp(std::log(x0) + std::log(x1 / x0) * U(r)), u = (double)(r() >> 11) * 0x1p-53;
        const double v = cs::angle_icdf_v(u, x), s = cs::sigma_ratio(x);
        const Q T = tail(2, x), vt = root((Q)(1.0 - u) * T, x, v), st = 3 * T / 8;
        const double ev = (double)((v - vt) / vt), es = (double)((s - st) / st);
        sv += ev * ev;
        ss += es * es;
    }
    std::printf("%.6e %.6e\n", std::sqrt(sv / n), std::sqrt(ss / n));
}
"""


def _host_code(name):
    t = open(os.path.join(CSRC, name)).read()
    t = re.sub(r'asm volatile\(""[^;]*;', "", t)
    t = re.sub(r'double r;\s*asm\("v_fma_f64[^;]*;\s*return r;', "return fma(a, b, c);", t)
    t = re.sub(r'uint32_t r;\s*asm\("v_bitop3[^;]*;\s*return r;', "return a ^ b ^ c;", t)
    t = t.replace("const __attribute__((address_space(4))) double*", "const double*")
    t = t.replace("__attribute__((noinline))", "inline").replace("(cdptr)", "").replace("#pragma once", "")
    t = t.replace("return __builtin_amdgcn_ballot_w64(p);", "return p ? 1 : 0;")
    for a, b in (("rcpf(", "rcp32("), ("rcp(", "rcp64("), ("rsq(", "rsq64("), ("logf(", "log32("), ("exp2f(", "exp32("),
                 ("fmed3f(", "med3("), ("frexp_mant(", "frexp_m("), ("frexp_exp(", "frexp_e(")):
        t = t.replace("__builtin_amdgcn_" + a, b)
    return re.sub(r'#include "(cs_\w+\.h)"', lambda m: _host_code(m.group(1)), re.sub(r"#include <.*>", "", t))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("sampler")
    (d / "m.cpp").write_text(SHIM + _host_code("cs_device.h") + MAIN)
    subprocess.run(["g++", "-O2", "-std=gnu++17", "-ffp-contract=off", "-mfma", str(d / "m.cpp"), "-o", str(d / "m")],
                   check=True)

    def run(x0, x1, n=100000):
        out = subprocess.run([str(d / "m"), repr(x0), repr(x1), str(n)], check=True, capture_output=True, text=True)
        return [float(v) for v in out.stdout.split()]

    return run


@pytest.mark.parametrize("x0, x1, bound", [
    (1e-8, 1e-3, 2.30e-16), (1e-3, 2.0 ** -8, 2.30e-16), (2.0 ** -8, 0.03, 2.32e-16), (0.03, 0.1, 2.41e-16),
    (0.1, 0.15, 2.80e-16), (0.15, 0.5, 2.81e-16), (0.5, 1.0, 3.10e-16), (1.0, 10.0, 3.80e-16),
    (10.0, 100.0, 4.41e-16), (100.0, 1e3, 6.01e-16), (1e3, 1e4, 7.60e-16), (1e4, 2.0 ** 17, 9.80e-16),
    (2.0 ** 17, 1e9, 1.75e-15)])
def test_root_error(model, x0, x1, bound):
    assert model(x0, x1)[0] <= bound


@pytest.mark.parametrize("x0, x1, bound", [(2.0 ** -20, 2.0 ** 17, 7.0e-17), (2.0 ** 17, 1e6, 1.09e-16),
                                           (1e6, 1e9, 1.12e-16), (1e9, 1e15, 1.07e-16)])
def test_cross_section_error(model, x0, x1, bound):
    assert model(x0, x1)[1] <= bound
