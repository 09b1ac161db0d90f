"""Writes cs_icdf_table.h: the polynomials of the plain sampler
(angle_icdf_v in cs_device.h).

    python paper_2206_02937_amd/csrc/gen_icdf_table.py

kTailPoly   P(sigma) = sum_k 2 sigma^k / (2k + 3) on [0, 1/4], degree 15: the
            Chebyshev interpolant (its nearest singularity, sigma = 1, is 7
            half-widths from the centre, so the error falls by 13.9 per
            degree), computed at 60 digits and rounded to double; the script
            refuses to write it if the rounded polynomial is off by more than
            1.5e-17 relative (beyond the rounding of its leading term).
kSmallZ     (8/3) s(x) about x = 0 to x^7, for x < 2^-8 (the next term is
            below 2e-17 there).
kMidZ       the same for 2^-8 <= x < 1/8, in powers of x - kMidC: the Chebyshev
            interpolant (its nearest singularity, x = -1/2, is 9.3 half-widths
            from the centre, so the error falls by 18.6 per degree); kMidC, near
            the middle, is where the leading coefficient is a double to 1e-18.
kStart*     FP32 starting values of the root, fitted to the exact inverse by
            reweighted least squares (about minimax in the relative error of
            v): with w = 1 - u, L = ln(1 + 2x), t = L / (L + 2),
              h(w, t) = ln(1 + x v) / (L w) = sum_j t^j row_j(w)
            over 0 <= x <= 1000 (relative error of v 1e-2), and
              v / w = A(w) + x B(w)
            over 0 <= x < 2^-8 (8e-4), and P once more to FP32 accuracy.  They
            have to be good enough for one FP32 step (of third order, and of
            second for the small x) to reach about 1e-6.
"""
import os

import mpmath as mp
import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(HERE, "cs_icdf_table.h")
TAIL_TERMS = 16
SMALL_Z_TERMS = 8
SMALL_X = 2.0 ** -8
MID_X, MID_C, MID_Z_TERMS = 0.125, 0.06666851043701172, 14
X_MAX = 1000.0
T_SHIFT = 2.0
ROWS = (5, 5, 5, 4, 3)  # degree in w of row j
SMALL_A, SMALL_B = 8, 2
START_TAIL_DEG = 5


def tail_poly():
    """Monomial coefficients of the Chebyshev interpolant of P on [0, 1/4]."""
    n = TAIL_TERMS
    h = mp.mpf(1) / 8

    def p(s):
        return mp.nsum(lambda k: 2 * s ** k / (2 * k + 3), [0, 120]) if s else mp.mpf(2) / 3

    nodes = [h * (1 + mp.cos(mp.pi * (2 * i + 1) / (2 * n))) for i in range(n)]
    a = mp.matrix(n, n)
    b = mp.matrix(n, 1)
    for i, s in enumerate(nodes):
        b[i] = sum(2 * s ** k / (2 * k + 3) for k in range(140))
        for k in range(n):
            a[i, k] = s ** k
    c = mp.lu_solve(a, b)
    dbl = [float(v) for v in c]
    lead = mp.mpf(dbl[0]) - mp.mpf(2) / 3
    for i in range(200):
        s = mp.mpf(i) / 199 / 4
        exact = sum(2 * s ** k / (2 * k + 3) for k in range(140))
        got = sum(mp.mpf(v) * s ** k for k, v in enumerate(dbl)) - lead
        assert abs(got - exact) / exact < mp.mpf("1.5e-17"), (s, float((got - exact) / exact))
    return dbl


def total(x):
    """(8/3) s(x), closed form (use at 60 digits)."""
    l = mp.log1p(2 * x)
    return mp.mpf(2) * ((1 + x) / x ** 3 * (2 * x * (1 + x) / (1 + 2 * x) - l) + l / (2 * x)
                        - (1 + 3 * x) / (1 + 2 * x) ** 2)


def mid_z():
    n, lo, hi, c = MID_Z_TERMS, mp.mpf(SMALL_X), mp.mpf(MID_X), mp.mpf(MID_C)
    nodes = [(lo + hi) / 2 + (hi - lo) / 2 * mp.cos(mp.pi * (2 * i + 1) / (2 * n)) for i in range(n)]
    a, b = mp.matrix(n, n), mp.matrix(n, 1)
    for i, x in enumerate(nodes):
        b[i] = total(x)
        for k in range(n):
            a[i, k] = (x - c) ** k
    out = [float(v) for v in mp.lu_solve(a, b)]
    for i in range(300):
        x = lo + (hi - lo) * i / 299
        got = sum(mp.mpf(v) * (x - c) ** k for k, v in enumerate(out))
        assert abs(got / total(x) - 1) < mp.mpf("4e-17"), (float(x), float(got / total(x) - 1))
    return out


def small_z():
    # (8/3) s(x) = int_0^2 f dv with f expanded in x: a^-m = sum binom(-m, k) (x v)^k
    out = []
    for k in range(SMALL_Z_TERMS):
        c3, c2, c1 = mp.binomial(-3, k), mp.binomial(-2, k), mp.binomial(-1, k)
        v = mp.mpf(2)
        out.append((c3 + c1) * v ** (k + 1) / (k + 1) - c2 * (2 * v ** (k + 2) / (k + 2) - v ** (k + 3) / (k + 3)))
    x = mp.mpf(SMALL_X)
    got = sum(c * x ** k for k, c in enumerate(out))
    assert abs(got / total(x) - 1) < mp.mpf("1e-16"), float(got / total(x) - 1)
    return [float(c) for c in out]


_GX, _GW = np.polynomial.legendre.leggauss(40)


def _tail(v, x):
    top, tot = np.log1p(x * v), 0.0
    for t, w in zip(0.5 * (_GX + 1.0), 0.5 * _GW):
        s = top * t
        a, y = np.exp(s), np.expm1(s) / x
        tot = tot + w * (a ** -3 + 1.0 / a - y * (2.0 - y) / (a * a)) * a
    return tot * top / x


def _icdf(w, x):
    target = w * _tail(np.full_like(x, 2.0), x)
    lo, hi = np.zeros_like(x), np.full_like(x, 2.0)
    for _ in range(56):
        mid = 0.5 * (lo + hi)
        above = _tail(mid, x) > target
        hi, lo = np.where(above, mid, hi), np.where(above, lo, mid)
    return 0.5 * (lo + hi)


def _cheb(n):
    return 0.5 * (np.cos(np.pi * (np.arange(n) + 0.5) / n) + 1.0)


def _fit(basis, y, weight):
    a, b = basis * weight[:, None], y * weight
    ww, best = np.ones_like(b), None
    for _ in range(60):
        c = np.linalg.lstsq(a * ww[:, None], b * ww, rcond=None)[0]
        e = np.abs(a @ c - b)
        if best is None or e.max() < best[0]:
            best = (e.max(), c)
        ww *= (0.3 + e / e.max()) ** 0.5
        ww /= ww.max()
    return best


def start_rows():
    top = np.log1p(2 * X_MAX)
    tm = top / (top + T_SHIFT)
    t = tm * _cheb(48)
    w, L = [a.ravel() for a in np.meshgrid(_cheb(56), T_SHIFT * t / (1 - t), indexing="ij")]
    x = np.expm1(L) / 2
    v = _icdf(w, x)
    h = np.log1p(x * v) / L / w
    tt = L / (L + T_SHIFT)
    basis = np.stack([w ** i * tt ** j for j, n in enumerate(ROWS) for i in range(n + 1)], 1)
    err, c = _fit(basis, h, (1 + x * v) * L * w / (x * v))
    assert err < 1.2e-2, err
    rows, i = [], 0
    for n in ROWS:
        rows.append(c[i:i + n + 1])
        i += n + 1
    return err, rows


def start_small():
    w, x = [a.ravel() for a in np.meshgrid(_cheb(64), 1e-9 + (SMALL_X - 1e-9) * _cheb(8), indexing="ij")]
    v = _icdf(w, x)
    basis = np.stack([w ** i for i in range(SMALL_A + 1)] + [x * w ** i for i in range(SMALL_B + 1)], 1)
    err, c = _fit(basis, v / w, w / v)
    assert err < 8e-4, err
    return err, c[:SMALL_A + 1], c[SMALL_A + 1:]


def start_tail():
    s = 0.25 * _cheb(64)
    p = np.sum(2.0 * s[:, None] ** np.arange(80) / (2.0 * np.arange(80) + 3.0), 1)
    err, c = _fit(s[:, None] ** np.arange(START_TAIL_DEG + 1), p, 1.0 / p)
    assert err < 1e-7, err
    return err, c


def main():
    mp.mp.dps = 60
    tail, sz, mz = tail_poly(), small_z(), mid_z()
    e_rows, rows = start_rows()
    e_small, a, b = start_small()
    e_tail, pt = start_tail()
    width = max(len(r) for r in rows)
    f = lambda vals: ", ".join("%.7ef" % v for v in vals)  # noqa: E731
    lines = [
        "// Generated by gen_icdf_table.py: polynomials of the plain sampler.",
        "#pragma once",
        "",
        "namespace cs {",
        "",
        "// P(sigma) = sum_k 2 sigma^k / (2k + 3) on [0, 1/4]",
        f"constexpr int kTailPolyTerms = {TAIL_TERMS};",
        f"__constant__ constexpr double kTailPoly[{TAIL_TERMS}] = {{",
        *["    %.17e," % v for v in tail],
        "};",
        "",
        "// (8/3) s(x) about x = 0, for x < kSmallX",
        f"constexpr double kSmallX = {SMALL_X!r};",
        f"constexpr int kSmallZTerms = {SMALL_Z_TERMS};",
        f"__constant__ constexpr double kSmallZ[{SMALL_Z_TERMS}] = {{",
        *["    %.17e," % v for v in sz],
        "};",
        "",
        "// the same in powers of x - kMidC, for kSmallX <= x < kMidX",
        f"constexpr double kMidX = {MID_X!r}, kMidC = {MID_C!r};",
        f"constexpr int kMidZTerms = {MID_Z_TERMS};",
        f"__constant__ constexpr double kMidZ[{MID_Z_TERMS}] = {{",
        *["    %.17e," % v for v in mz],
        "};",
        "",
        f"// h(w, t), t = L / (L + kStartShift): relative error of v {e_rows:.1e}",
        f"constexpr float kStartShift = {T_SHIFT}f;",
        f"constexpr int kStartRows = {len(rows)};",
        f"constexpr int kStartDeg[{len(rows)}] = {{{', '.join(str(len(r) - 1) for r in rows)}}};",
        f"constexpr float kStart[{len(rows)}][{width}] = {{",
        *["    {" + f(list(r) + [0.0] * (width - len(r))) + "}," for r in rows],
        "};",
        "",
        f"// v / w for x < kSmallX: A(w) + x B(w), relative error {e_small:.1e}",
        f"constexpr int kStartSmallA = {SMALL_A}, kStartSmallB = {SMALL_B};",
        f"constexpr float kStartA[{SMALL_A + 1}] = {{{f(a)}}};",
        f"constexpr float kStartB[{SMALL_B + 1}] = {{{f(b)}}};",
        "",
        f"// P(sigma) on [0, 1/4] in FP32, relative error {e_tail:.1e}",
        f"constexpr int kStartTailDeg = {START_TAIL_DEG};",
        f"constexpr float kStartTail[{START_TAIL_DEG + 1}] = {{{f(pt)}}};",
        "",
        "}  // namespace cs",
        "",
    ]
    with open(OUT, "w") as fh:
        fh.write("\n".join(lines))


if __name__ == "__main__":
    main()
