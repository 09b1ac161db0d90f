// cs_device.h -- device-side arithmetic of the Compton step for gfx950.
//
// Counter-based random numbers, the in-cell pairing bijection, the
// Klein-Nishina cross-section and angular CDF, the inverse-CDF sampler and
// the rest-frame/lab kinematics.  All physics arithmetic is FP64 and written
// in forms free of catastrophic cancellation for gamma >> 1 (the Lorentz
// boosts and back-transforms), so that a FP32-stored plasma loses nothing
// beyond its storage rounding.
//
// Units: momenta in m_e c, energies in m_e c^2, s(x) = sigma_KN / sigma_T.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cs_icdf_table.h"
#include "cs_sigma_table.h"

namespace cs {

// The lanes in which a comparison holds, and whether it holds in any: scalar
// tests of the compare's mask.  Masks of several conditions are combined as
// scalars (a combined condition would pass through a vector register).
__device__ __forceinline__ uint64_t lanes(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool any_lane(bool p) { return lanes(p) != 0; }

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of the 4x32
// S-box, key advanced by the Weyl constants between rounds.
// ---------------------------------------------------------------------------
struct u32x4 {
    uint32_t a, b, c, d;
};

// a ^ b ^ c in one v_bitop3_b32 (truth table 0x96); c must be wave-uniform
// (it is read from a scalar register).
__device__ __forceinline__ uint32_t xor3_uniform(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

// The key (k0, k1) must be wave-uniform (it is the seed everywhere here).
__device__ __forceinline__ u32x4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                          uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t m0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t m1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3_uniform((uint32_t)(m1 >> 32), c1, k0);
        const uint32_t n2 = xor3_uniform((uint32_t)(m0 >> 32), c3, k1);
        c1 = (uint32_t)m1;
        c3 = (uint32_t)m0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return {c0, c1, c2, c3};
}

// Stream purposes (fourth counter word, low byte).
enum : uint32_t {
    kPair = 1,
    kCollide = 2,
    kScatter = 3,
    // no-time-counter candidate selection
    kNtcCount = 4,
    kNtcPick = 5,
    kNtcScatter = 6,
    kNtcWeight = 7
};

// counter = (index lo, index hi, step lo, step hi << 8 | purpose), key = seed.
__device__ __forceinline__ u32x4 draw(uint64_t seed, uint64_t index, uint64_t step, uint32_t purpose) {
    return philox10((uint32_t)index, (uint32_t)(index >> 32), (uint32_t)step,
                    ((uint32_t)(step >> 32) << 8) | purpose, (uint32_t)seed, (uint32_t)(seed >> 32));
}

// 53-bit uniform in [0, 1): top 27 bits of a, top 26 bits of b.
__device__ __forceinline__ double uniform53(uint32_t a, uint32_t b) {
    return fma((double)(a >> 5), 67108864.0, (double)(b >> 6)) * 0x1p-53;
}

// ---------------------------------------------------------------------------
// In-cell pairing: 4-round Feistel network over b = ceil(log2 M) bits with
// cycle-walking into [0, M) (Black & Rogaway 2002).  The left part has
// floor(b/2) bits and the right part the rest; a round maps (L, R) to
// (R, L ^ F(R)), so the widths trade places each round and are back after
// four.  Round function: MurmurHash3's 32-bit finaliser of (right part ^ key
// word), cut to the width of the left part.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t fmix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

struct FeistelKey {
    uint32_t k[4];
    uint32_t bits;  // b = ceil(log2 M)
};

__device__ __forceinline__ uint32_t ceil_log2(uint32_t M) { return M <= 1 ? 0u : 32u - __clz(M - 1u); }

// One pass of the network: the permutation of [0, 2^b) at v.
__device__ __forceinline__ uint32_t feistel(uint32_t v, const FeistelKey& key) {
    const uint32_t a = key.bits >> 1, c = key.bits - a;
    const uint32_t mask_a = (1u << a) - 1u, mask_c = (1u << c) - 1u;
    uint32_t L = v >> c, R = v & mask_c;  // widths a, c
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
        const uint32_t R1 = L ^ (fmix32(R ^ key.k[r]) & mask_a);  // (L, R) -> (R, R1): widths c, a
        const uint32_t R2 = R ^ (fmix32(R1 ^ key.k[r + 1]) & mask_c);  // -> (R1, R2): widths a, c
        L = R1;
        R = R2;
    }
    return (L << c) | R;
}

// The cycle-walk always ends: i lies on a cycle of the permutation of
// [0, 2^b), and that cycle returns to i, which is < M.
__device__ __forceinline__ uint32_t shuffle_index(uint32_t i, uint32_t M, const FeistelKey& key) {
    if (M <= 1u) return 0u;
    uint32_t v = i;
    do {
        v = feistel(v, key);
    } while (v >= M);
    return v;
}

// ---------------------------------------------------------------------------
// Klein-Nishina.  With a = 1 + x(1 - mu) the rest-frame angular density is
// f(mu) = a^-3 + a^-1 - (1 - mu^2) a^-2 (unnormalised), and
// s(x) = (3/8) int_{-1}^{1} f dmu.
// ---------------------------------------------------------------------------

// Upper tail of the angular integral, T(v) = int_{1-v}^{1} f dmu, by the
// three integrals in w = 1 - mu (a = 1 + x w; z = x v, A = 1 + z):
//   int a^-3 dw = v (2 + z) / (2 A^2),
//   int a^-1 dw = log1p(z) / x,
//   int w (2 - w) a^-2 dw = 2 phi2(z) / x^2 - phi3(z) / x^3,
//     phi2 = log1p(z) - z / (1 + z),  phi3 = z - 2 log1p(z) + z / (1 + z),
// and T = first + second - third.  With s = z / (2 + z) (so log1p(z) =
// 2 atanh(s)), q = s / x = v / (2 + z) and sigma = s^2,
//   log1p(z) = 2 s (1 + sigma P / 2),  P = sum_{k>=0} 2 sigma^k / (2k + 3),
// and the powers of z cancel in closed form:
//   T = v (2 + z) / (2 A^2) + q (2 - v (2 - v) / A) + q^3 (x^2 - 2x - 2) P.
// One series of positive terms is all that is left of the logarithm (three
// before, for the integrals one by one), nothing cancels by more than a factor
// of two at any x, and the form holds down to x = 0.  It serves z < 2
// (sigma < 1/4), with P the degree-15 polynomial of cs_icdf_table.h; above,
// the logarithm itself is formed and the integrals are taken as they stand
// (z >= 2 needs x >= 1, where they do not cancel).

typedef const __attribute__((address_space(4))) double* cdptr;  // constant (scalar-load) space

// a * b + c with c held in a scalar register pair: one v_fma_f64 that reads
// the coefficient directly (the compiler's own selection copies each scalar
// coefficient into vector registers first, two extra instructions per term).
__device__ __forceinline__ double fma_sgpr(double a, double b, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

// 1/a to about an ulp (hardware estimate and two Newton steps).
__device__ __forceinline__ double recip_approx(double a) {
    double r = __builtin_amdgcn_rcp(a);
    r = fma(fma(-a, r, 1.0), r, r);
    return fma(fma(-a, r, 1.0), r, r);
}


// P(sigma) for 0 <= sigma < 1/4.  sigma <= 1.5e-3: the first six terms of
// the series (remainder below 1e-17), else the degree-15 polynomial in two
// interleaved Horner chains.  Which form a lane takes depends on its own
// sigma only, so its bits do not depend on the lanes that share its wave; a
// wave whose lanes are all small skips the longer form.  The coefficient
// pointer passes through an empty asm so that the coefficients are read with
// scalar loads at each use instead of being held in vector registers.
__device__ __forceinline__ double tail_poly(double sg) {
    const bool low = sg <= 1.5e-3;
    double p = 2.0 / 3.0;
    if (any_lane(low)) {
        double t = 2.0 / 13.0;
        t = fma_sgpr(t, sg, 2.0 / 11.0);
        t = fma_sgpr(t, sg, 2.0 / 9.0);
        t = fma_sgpr(t, sg, 2.0 / 7.0);
        t = fma_sgpr(t, sg, 2.0 / 5.0);
        p = fma_sgpr(t, sg, 2.0 / 3.0);
    }
    if (any_lane(!low)) {
        cdptr c = (cdptr)kTailPoly;
        asm volatile("" : "+s"(c));
        static_assert(kTailPolyTerms % 2 == 0, "two chains of equal length");
        const double s2 = sg * sg;
        double e = c[kTailPolyTerms - 2], o = c[kTailPolyTerms - 1];
#pragma unroll
        for (int k = kTailPolyTerms - 4; k >= 0; k -= 2) {
            e = fma_sgpr(e, s2, c[k]);
            o = fma_sgpr(o, s2, c[k + 1]);
        }
        const double h = fma(o, sg, e);
        if (!low) p = h;
    }
    return p;
}

// T(v) at x, with what the density at v needs besides: iA = 1 / (1 + x v)
// and w = v (2 - v).  One reciprocal serves 1/A and the argument of the
// series: for z < 2 of s = z / (2 + z), above of (m - 1) / (m + 1) with
// A = 2^k m, m in [1/sqrt 2, sqrt 2), whose logarithm takes the same P.
// ANY_BIG = false: for waves without a lane of z >= 2 (the same arithmetic
// for the others).  ROUND: where z >= 2, every operation rounded (what the
// shipped network's training targets, x up to 1e3, were made with), or two
// roundings fewer, or these above kTailFusedX, where the root takes up more of
// them.
struct KnTail {
    double T, iA, w;
};

enum TailRound { kTailPlain, kTailFused, kTailByX };
constexpr double kTailFusedX = 1e3;

template <bool ANY_BIG, TailRound ROUND>
__device__ __forceinline__ KnTail kn_tail_z(double v, double x, double z, bool big) {
    const double t2 = z + 2.0, A = z + 1.0;
    double num = z, den = t2, k = 0.0;
    if (ANY_BIG && big) {
        const double m0 = __builtin_amdgcn_frexp_mant(A);  // [1/2, 1)
        const bool low = m0 < 0.70710678118654757;
        const double m = low ? m0 + m0 : m0;
        k = (double)(__builtin_amdgcn_frexp_exp(A) - (low ? 1 : 0));
        num = m - 1.0;
        den = m + 1.0;
    }
    // one hardware estimate for both reciprocals, the last Newton step on each
    const double dA = den * A;
    double rr = __builtin_amdgcn_rcp(dA);
    rr = fma(fma(-dA, rr, 1.0), rr, rr);
    const double r0 = rr * A, i0 = rr * den;
    const double r = fma(fma(-den, r0, 1.0), r0, r0);
    KnTail o;
    o.iA = fma(fma(-A, i0, 1.0), i0, i0);
    o.w = fma(-v, v, v + v);
    const double s = num * r, sg = s * s;
    const double P = tail_poly(sg);
    const double first = 0.5 * v * (t2 * o.iA) * o.iA;
    if (!(ANY_BIG && big)) {
        const double q = v * r;
        const double c = fma(x, x - 2.0, -2.0);
        o.T = fma(q, fma(-o.w, o.iA, 2.0), fma(q * q * q, P * c, first));
    } else {
        // ln A = k ln 2 + 2 atanh(s); ln 2 as its leading 32 bits and the rest
        const double l = s * fma(sg, P, 2.0);
        const double lnA = fma(k, 0x1.62e42feep-1, fma(k, 0x1.a39ef35793c76p-33, l));
        const double ix = recip_approx(x), zA = z * o.iA;
        const double phi2 = lnA - zA, phi3 = (z - 2.0 * lnA) + zA;
        const double y = 2.0 * phi2 - phi3 * ix;
        const double plain = first + ix * (lnA - ix * y), fused = fma(ix, fma(-ix, y, lnA), first);
        o.T = ROUND == kTailPlain ? plain : (ROUND == kTailFused || x > kTailFusedX ? fused : plain);
    }
    return o;
}

template <TailRound ROUND = kTailPlain>
__device__ __forceinline__ KnTail kn_tail(double v, double x) {
    const double z = x * v;
    const bool big = z >= 2.0;
    if (any_lane(big)) return kn_tail_z<true, ROUND>(v, x, z, big);
    return kn_tail_z<false, ROUND>(v, x, z, false);
}

// s(x) = sigma_KN(x) / sigma_T.  Below 2: the per-segment Taylor polynomial
// of cs_sigma_table.h, evaluated per lane (each lane loads its own segment's
// 12 coefficients; no lane waits for another's branch).  `tab` is kSigTab or
// a copy of it (e.g. in LDS): the same coefficients, the same result.  From
// 2 to 2^17 the second table (segment index and centre from the exponent and
// the top four mantissa bits); above, the whole angular integral (3/8) T(2),
// whose coefficients come by scalar loads (log1p's, held in vector registers
// across the pair kernel's loop, cost it a wave per SIMD).
__device__ __forceinline__ double sigma_ratio_tab(double x, const double* tab) {
    if (x < kSigTabMax) {
        int j = (int)(x * kSigTabInvWidth);
        j = j < 0 ? 0 : (j > kSigTabSegments - 1 ? kSigTabSegments - 1 : j);
        const double t = x - ((double)j + 0.5) / kSigTabInvWidth;
        const double* a = tab + j * kSigTabTerms;
        double acc = a[kSigTabTerms - 1];
#pragma unroll
        for (int n = kSigTabTerms - 2; n >= 0; --n) acc = fma(acc, t, a[n]);
        return acc;
    }
    if (x < kSigTabHiMax) {
        // (hi >> 16) = (1023 + e) << 4 | m for x = 2^e (1 + m/16 + ...)
        const int hi = __double2hiint(x);
        const int j = (hi >> 16) - ((1023 + 1) << 4);
        const double t = x - __hiloint2double((hi & (int)0xFFFF0000) | 0x8000, 0);
        const double* a = kSigTabHi + j * kSigTabTerms;
        double acc = a[kSigTabTerms - 1];
#pragma unroll
        for (int n = kSigTabTerms - 2; n >= 0; --n) acc = fma(acc, t, a[n]);
        return acc;
    }
    return 0.375 * kn_tail<kTailFused>(2.0, x).T;
}

__device__ __forceinline__ double sigma_ratio(double x) { return sigma_ratio_tab(x, kSigTab); }

// (8/3) s(x) = T(2): the whole angular integral.  Below kMidX as polynomials in
// x, whose rounding takes 0.7e-16 of it (rms), where the tail itself loses 1.7e-16 (with
// which the sampled v was 2.5e-16 off, for x in [2^-8, 0.1); 1.9e-16 so).  Above, the
// tail's rounding errors at 2 and at v are partly the same.
__device__ __forceinline__ double kn_total(double x) {
    if (x < kSmallX) {
        double z = kSmallZ[kSmallZTerms - 1];
#pragma unroll
        for (int k = kSmallZTerms - 2; k >= 0; --k) z = fma_sgpr(z, x, kSmallZ[k]);
        return z;
    }
    if (x < kMidX) {
        cdptr c = (cdptr)kMidZ;
        asm volatile("" : "+s"(c));
        static_assert(kMidZTerms % 2 == 0, "two chains of equal length");
        const double t = x - kMidC, t2 = t * t;
        double e = c[kMidZTerms - 2], o = c[kMidZTerms - 1];
#pragma unroll
        for (int k = kMidZTerms - 4; k >= 0; k -= 2) {
            e = fma_sgpr(e, t2, c[k]);
            o = fma_sgpr(o, t2, c[k + 1]);
        }
        return fma(o, t, e);
    }
    return kn_tail(2.0, x).T;
}

// FP32 Horner chain with compile-time coefficients, degree D.
template <int D>
__device__ __forceinline__ float horner_f32(const float (&c)[D + 1], float t) {
    float a = c[D];
#pragma unroll
    for (int k = D - 1; k >= 0; --k) a = fmaf(a, t, c[k]);
    return a;
}

// Row j of the starting value's polynomial at w.
template <int J>
__device__ __forceinline__ float start_row(float w) {
    float a = kStart[J][kStartDeg[J]];
#pragma unroll
    for (int k = kStartDeg[J] - 1; k >= 0; --k) a = fmaf(a, w, kStart[J][k]);
    return a;
}

// The root v of T(v) = target to about 1e-6 in FP32, for kSmallX <= x: the
// polynomial starting value (1e-2), then one Halley step on the FP32 tail.
__device__ __forceinline__ float icdf_start(float w, float x, float target) {
    const float lx = x < 0.03f ? fmaf(x, fmaf(x, 2.6666667f, -2.0f), 2.0f)
                               : 0.69314718f * __builtin_amdgcn_logf(fmaf(2.0f, x, 1.0f)) * __builtin_amdgcn_rcpf(x);
    const float L = lx * x;  // ln(1 + 2x)
    const float t = L * __builtin_amdgcn_rcpf(L + kStartShift);
    static_assert(kStartRows == 5, "rows");
    float h = start_row<4>(w);
    h = fmaf(h, t, start_row<3>(w));
    h = fmaf(h, t, start_row<2>(w));
    h = fmaf(h, t, start_row<1>(w));
    h = fmaf(h, t, start_row<0>(w));
    h *= w;
    const float y = h * L;  // ln(1 + x v); v = (e^y - 1) / x
    float v = y < 0.25f ? h * lx * fmaf(y, fmaf(y, fmaf(y, 0.041666668f, 0.16666667f), 0.5f), 1.0f)
                        : (__builtin_amdgcn_exp2f(1.44269504f * y) - 1.0f) * __builtin_amdgcn_rcpf(x);
    v = fminf(v, 2.0f);
    const float z = x * v, t2 = z + 2.0f, A = z + 1.0f;
    const float rr = __builtin_amdgcn_rcpf(t2 * A);
    const float r = rr * A, iA = rr * t2;
    const float wv = fmaf(-v, v, v + v);
    const float first = 0.5f * v * (t2 * iA) * iA;
    float T;
    if (z < 2.0f) {
        const float s = z * r, sg = s * s, q = v * r;
        const float P = horner_f32<kStartTailDeg>(kStartTail, sg);
        T = first + q * fmaf(-wv, iA, 2.0f) + (q * q * q) * (P * fmaf(x, x - 2.0f, -2.0f));
    } else {
        const float lnA = 0.69314718f * __builtin_amdgcn_logf(A);
        const float ix = __builtin_amdgcn_rcpf(x), zA = z * iA;
        T = first + ix * (lnA - ix * (2.0f * (lnA - zA) - ((z - 2.0f * lnA) + zA) * ix));
    }
    const float R = T - target;
    const float f = iA * fmaf(iA, iA - wv, 1.0f);
    const float g = fmaf(x, fmaf(iA, fmaf(3.0f, iA, -2.0f * wv), 1.0f), 2.0f - 2.0f * v);  // f' = -iA^2 g
    return v - 2.0f * R * f * __builtin_amdgcn_rcpf(fmaf(R * iA * iA, g, 2.0f * f * f));
}

// The same for x < kSmallX: starting value w (A(w) + x B(w)) (8e-4), then a
// Newton step on the tail and its density as polynomials to second order in x.
__device__ __forceinline__ float icdf_start_small(float w, float x, float target) {
    float v = w * fmaf(x, horner_f32<kStartSmallB>(kStartB, w), horner_f32<kStartSmallA>(kStartA, w));
    v = fminf(v, 2.0f);
    const float wv = fmaf(-v, v, v + v);
    const float xv = x * v;
    const float t0 = fmaf(v, fmaf(v, 0.33333333f, -1.0f), 2.0f);
    const float t1 = fmaf(v, fmaf(v, -0.5f, 1.3333333f), -2.0f);
    const float tq = fmaf(v, fmaf(v, 0.6f, -1.5f), 2.3333333f);
    const float R = fmaf(v, fmaf(xv, fmaf(xv, tq, t1), t0), -target);
    const float f = fmaf(xv, fmaf(2.0f, wv, -4.0f), 2.0f - wv);
    return fmaf(-R, __builtin_amdgcn_rcpf(f), v);
}

// One step of third order in FP64 from v towards the root of T(v) = target:
// d = R / f (R the residual, f the density), v - d (1 + d f' / (2 f)).
struct IcdfStep {
    double R, d, c2;  // residual, Newton step, d f' / (2 f)
};

template <TailRound ROUND = kTailPlain>
__device__ __forceinline__ IcdfStep icdf_step(double v, double x, double target) {
    const KnTail t = kn_tail<ROUND>(v, x);
    const double a2 = t.iA * t.iA;
    const double h = fma(-t.iA, t.w, 1.0 + a2);
    const double f = t.iA * h;
    double rf = __builtin_amdgcn_rcp(f);
    rf = fma(fma(-f, rf, 1.0), rf, rf);
    IcdfStep s;
    s.R = t.T - target;
    s.d = s.R * rf;
    // f' = -iA^2 (2 - 2v + x (1 + iA (3 iA - 2 w)))
    const double g = fma(x, fma(2.0, h, a2 - 1.0), fma(-2.0, v, 2.0));
    s.c2 = (-0.5 * s.d) * (a2 * (g * rf));
    return s;
}

// More steps where one did not settle it, safeguarded by a bisection bracket
// (a start far off), and every x above kTailFusedX, target and residual with
// the fewer roundings (x in [1e3, 1e4): v 7.7e-16 -> 6.9e-16 off, rms).
__device__ __attribute__((noinline)) double icdf_refine(double v, double x, double w1, double target) {
    double lo = 0.0, hi = 2.0;
    if (x > kTailFusedX) target = w1 * kn_tail<kTailFused>(2.0, x).T;
    for (int it = 0; it < 60; ++it) {
        const IcdfStep s = icdf_step<kTailByX>(v, x, target);
        double next = v - fma(s.d, fabs(s.c2) < 0.5 ? s.c2 : 0.0, s.d);
        if (fabs(s.d) <= 3e-6 * v) return next;
        if (s.R > 0.0)  // v too large
            hi = v;
        else
            lo = v;
        if (!(next > lo && next < hi)) next = 0.5 * (lo + hi);
        v = next;
        if (hi - lo <= 1e-16 * hi) break;
    }
    return v;
}

// Inverse CDF of the rest-frame scattering angle, returned as v = 1 - mu so
// that forward scatters (mu -> 1) keep relative precision: the v with
// tail(v) = (1 - u) Z, Z = tail(2) = (8/3) s(x).
//
// An FP32 start good to about 1e-6 (icdf_start: a fitted polynomial and one
// Halley step), then one step of third order on the FP64 residual.  A step
// below 3e-6 v ends the iteration, the error after it being about
// C v (3e-6)^3, C = O(1): round-off, which only the FP64 residual decides.
//
// What bounds it: VALU issue, about four cycles per wave and instruction in
// FP32 and FP64 alike, so the number of instructions counts, whatever their
// type: 420 per wave with x over [1e-8, 1e3] in every wave, 135 where all
// are below kSmallX, 731 over [1e3, 1e6], where icdf_refine answers.
// k_sample_plain on 2^22 FP32 samples of the first:
// 176.4 us with three series up to 30 terms for the tail below x = 1, its
// closed form above, and 2-4 FP64 Halley steps from the Thomson root;
// 44.7 us with this (22.6 us for the power-law plasma's inputs, 50.2 before).
// The two starts part at kSmallX because the cheap one needs the tail's
// expansion in x; the whole grid range on icdf_start alone would slow the
// small-x plasmas to its cost.
__device__ __forceinline__ double angle_icdf_v(double u, double x) {
    const double w1 = 1.0 - u;  // exact for u = k 2^-53
    const double target = w1 * kn_total(x);
    const float start = x < kSmallX ? icdf_start_small((float)w1, (float)x, (float)target)
                                    : icdf_start((float)w1, (float)x, (float)target);
    const double v = (double)__builtin_amdgcn_fmed3f(start, 0.0f, 2.0f);
    const IcdfStep s = icdf_step(v, x, target);
    double next = v - fma(s.d, s.c2, s.d);
    const bool settled = fabs(s.d) <= 3e-6 * v && x <= kTailFusedX;
    if (__builtin_expect(any_lane(!settled), 0)) {
        if (!settled) next = icdf_refine(v, x, w1, target);
    }
    return fmin(next, 2.0);
}

// ---------------------------------------------------------------------------
// Kinematics (FP64, cancellation-free forms)
// ---------------------------------------------------------------------------
struct d3 {
    double x, y, z;
};

__device__ __forceinline__ double dot(d3 a, d3 b) { return fma(a.x, b.x, fma(a.y, b.y, a.z * b.z)); }
__device__ __forceinline__ d3 cross(d3 a, d3 b) {
    return {fma(a.y, b.z, -(a.z * b.y)), fma(a.z, b.x, -(a.x * b.z)), fma(a.x, b.y, -(a.y * b.x))};
}
__device__ __forceinline__ d3 axpy(double a, d3 x, d3 y) { return {fma(a, x.x, y.x), fma(a, x.y, y.y), fma(a, x.z, y.z)}; }
__device__ __forceinline__ d3 scale(double a, d3 x) { return {a * x.x, a * x.y, a * x.z}; }

// sqrt(a) for a normal, positive a: the hardware reciprocal square root
// refined by Goldschmidt's iteration with two residual corrections (within
// about an ulp; no scaling or special-case handling).
__device__ __forceinline__ double sqrt_normal(double a) {
    const double y = __builtin_amdgcn_rsq(a);
    double g = a * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    double d = fma(-g, g, a);
    g = fma(d, h, g);
    d = fma(-g, g, a);
    return fma(d, h, g);
}

// n / d for normal d: the hardware reciprocal refined by two Newton steps,
// the quotient, and one residual correction (within about an ulp).
__device__ __forceinline__ double div_normal(double n, double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    const double q = n * r;
    return fma(fma(-d, q, n), r, q);
}

struct XFlux {
    double x, flux;  // rest-frame photon energy x = gamma eps - p.k, flux = x / (gamma eps)
};

// gamma eps = sqrt((1 + p.p) k.k) (one square root); x = gamma eps - p.k, and
// for p.k > 0 the cancellation-free x = (k.k + |p x k|^2) / (gamma eps + p.k)
// (gamma^2 eps^2 - (p.k)^2 = eps^2 + |p x k|^2).  Both cases share one
// division: flux = num / den with (num, den) = (gamma eps - p.k, gamma eps),
// resp. (k.k + |p x k|^2, gamma eps (gamma eps + p.k)), and then x = flux
// gamma eps in the second case.  pp = p.p, kk = k.k.  FAST: the square root
// and the division are the refined hardware estimates above, valid while
// their operands are normal numbers.
template <bool FAST>
__device__ __forceinline__ XFlux x_flux_impl(d3 p, d3 k, double pp, double kk) {
    const double a = (1.0 + pp) * kk;
    const double ge = FAST ? sqrt_normal(a) : sqrt(a);
    const double pk = dot(p, k);
    const bool fwd = pk > 0.0;
    const d3 c = cross(p, k);
    const double num = fwd ? kk + dot(c, c) : ge - pk;
    const double den = fwd ? ge * (ge + pk) : ge;
    XFlux r;
    r.flux = FAST ? div_normal(num, den) : num / den;
    r.x = fwd ? r.flux * ge : num;
    return r;
}

// The range of a = (1 + p.p) k.k in which every operand of the fast form is
// normal.
constexpr double kFluxNormalMin = 1e-300, kFluxNormalMax = 1e300;

// The fast form there; the IEEE square root and division outside.
__device__ __forceinline__ XFlux x_flux(d3 p, d3 k, double pp, double kk) {
    if (kk == 0.0) return {0.0, 0.0};
    const double a = (1.0 + pp) * kk;
    if (a >= kFluxNormalMin && a <= kFluxNormalMax) return x_flux_impl<true>(p, k, pp, kk);
    return x_flux_impl<false>(p, k, pp, kk);
}

struct PairInv {
    double gamma, eps, x, flux;
};

__device__ __forceinline__ PairInv pair_invariants(d3 p, d3 k) {
    const double pp = dot(p, p), kk = dot(k, k);
    const XFlux xf = x_flux(p, k, pp, kk);
    PairInv r;
    r.gamma = sqrt(1.0 + pp);
    r.eps = sqrt(kk);
    r.x = xf.x;
    r.flux = xf.flux;
    return r;
}

struct Scattered {
    d3 p1, k1;
    double e_before, e_after;
};

// Resolve one collision.  Rest frame of the electron (velocity p/gamma):
// photon direction n from the decomposition of k along p_hat (perpendicular
// part unchanged, parallel part gamma k_par - |p| eps written without
// cancellation); scattered direction d = mu n + sin(theta)(cos(phi) e1 +
// sin(phi) e2) about the Duff et al. (JCGT 2017) orthonormal basis of n,
// with v = 1 - mu and sin(theta) = sqrt(v (2 - v));
// Compton shift x1 = x / (1 + x v); back-boost with the pre-collision
// p (parallel part x1 (gamma c + |p|), again cancellation-free); the
// electron takes p + k - k1.
__device__ __forceinline__ Scattered scatter(d3 p, d3 k, const PairInv& inv, double v, double u_phi) {
    const double gamma = inv.gamma, eps = inv.eps, x = inv.x;
    const double pp2 = dot(p, p);
    const double pp = sqrt(pp2);
    d3 n, ph;
    const bool moving = pp > 0.0;
    if (moving) {
        ph = scale(1.0 / pp, p);
        const double kpar = dot(k, ph);
        const d3 kperp = axpy(-kpar, ph, k);
        double kpar_r;
        if (kpar <= 0.0) {
            kpar_r = gamma * kpar - pp * eps;
        } else {
            const d3 c = cross(ph, k);
            kpar_r = (eps * eps - gamma * gamma * dot(c, c)) / (gamma * kpar + pp * eps);
        }
        n = axpy(kpar_r, ph, kperp);
    } else {
        ph = {0.0, 0.0, 0.0};
        n = k;
    }
    const double nn = 1.0 / sqrt(dot(n, n));
    n = scale(nn, n);
    // orthonormal basis (Duff et al. 2017)
    const double s = n.z >= 0.0 ? 1.0 : -1.0;
    const double a = -1.0 / (s + n.z);
    const double b = n.x * n.y * a;
    const d3 e1 = {1.0 + s * n.x * n.x * a, s * b, -s * n.x};
    const d3 e2 = {b, s + n.y * n.y * a, -n.y};
    double sphi, cphi;
    sincospi(2.0 * u_phi, &sphi, &cphi);
    const double mu = 1.0 - v;
    const double st = sqrt(v * (2.0 - v));
    d3 d = scale(mu, n);
    d = axpy(st * cphi, e1, d);
    d = axpy(st * sphi, e2, d);
    const double x1 = x / (1.0 + x * v);
    d3 k1;
    if (moving) {
        const double c = dot(d, ph);
        const d3 dperp = axpy(-c, ph, d);
        double par;
        if (c >= 0.0) {
            par = x1 * (gamma * c + pp);
        } else {
            const d3 cr = cross(ph, d);
            par = x1 * (1.0 - gamma * gamma * dot(cr, cr)) / (gamma * c - pp);
        }
        k1 = axpy(par, ph, scale(x1, dperp));
    } else {
        k1 = scale(x1, d);
    }
    Scattered r;
    r.k1 = k1;
    r.p1 = {(p.x + k.x) - k1.x, (p.y + k.y) - k1.y, (p.z + k.z) - k1.z};
    r.e_before = gamma + eps;
    r.e_after = sqrt(1.0 + dot(r.p1, r.p1)) + sqrt(dot(k1, k1));
    return r;
}

}  // namespace cs
