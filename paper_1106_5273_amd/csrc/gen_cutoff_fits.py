"""Generate cutoff_fits.h: polynomial fits used by the P2P kernels to evaluate
the Gaussian cutoff of Eq. (2) without cancellation, in float32 and in float64.

With s = rho / (sqrt(2) sigma) and x = s^2, the cutoff g of Eq. (2) and the
factor that enters dq/drho are the regularised lower incomplete gamma
functions P(3/2, x) = g and P(5/2, x) = g - (4 / (3 sqrt(pi))) s^3 exp(-x).

* s < 1 : P(a, x) = x^a e^{-x} / Gamma(a+1) * 1F1(1; a+1; x)  (all-positive
  Kummer series, no cancellation).  With M2(x) = 1F1(1; 7/2; x) we also have
  1F1(1; 5/2; x) = 1 + (2/5) x M2(x), so one fit of M2 on [0, 1] serves both.
* s >= 1 : 1 - P(3/2, x) = exp(-x) [erfcx(s) + (2/sqrt(pi)) s] and
  1 - P(5/2, x) = that + (4/(3 sqrt(pi))) s^3 exp(-x); erfcx(s) = u Pe(u) with
  u = 1/s in (0, 1] is fitted on s in [1, 6.3].  Beyond s ~ 6.1 the float32
  cutoff is exactly 1 and exp(-x) kills the (bounded) extrapolated fit.
  A relative error r of Pe changes P(3/2, x) and P(5/2, x) by
  exp(-x) erfcx(s) r, which falls like exp(-s^2) / s; the fit minimises that
  error relative to min(P(3/2, x), P(5/2, x)), so a low degree suffices.

The float64 form takes the same two functions over x < 3 and 3 <= x <= 43 (beyond
which both are 1 to double precision), M2 as sum_k x^k / Gamma(k + 7/2) and
Pe in t, which runs from -1 to 1 over u.

Fits are weighted least squares refined by iteratively reweighting toward
the minimax error (own fits, computed here from scipy's float64 special
functions as the reference, the float64 form's from mpmath's).  The exponential's
ln 2 is cut in two, of which the first times an integer below 2^12 is exact (Cody
and Waite, Software Manual for the Elementary Functions, 1980).
Run:  python gen_cutoff_fits.py
"""
import os

import mpmath as mp
import numpy as np
from scipy.special import erfcx, gammainc, hyp1f1

HERE = os.path.dirname(os.path.abspath(__file__))


def fit_rel(f, a, b, deg):
    t = np.linspace(a, b, 6000)
    y = f(t)
    V = np.vander(t, deg + 1, increasing=True)
    w = 1.0 / np.abs(y)
    c, *_ = np.linalg.lstsq(V * w[:, None], y * w, rcond=None)
    for _ in range(60):
        r = np.abs((V @ c - y) / y)
        w2 = w * np.sqrt(r / r.max()) + 1e-300
        c, *_ = np.linalg.lstsq(V * w2[:, None], y * w2, rcond=None)
    c32 = c.astype(np.float32)
    # float32 Horner error
    acc = np.full(t.shape, c32[-1], dtype=np.float32)
    t32 = t.astype(np.float32)
    for k in range(deg - 1, -1, -1):
        acc = (acc * t32 + c32[k]).astype(np.float32)
    err32 = np.abs((acc.astype(np.float64) - y) / y).max()
    return c32, np.abs((V @ c - y) / y).max(), err32


def fit_cutoff(s_lo, s_hi, deg):
    """erfcx(s) / u as a polynomial in u = 1/s, minimax in the relative error
    it causes in P(3/2, s^2) and P(5/2, s^2)."""
    s = np.linspace(s_lo, s_hi, 8000)
    u = 1.0 / s
    y = erfcx(s) / u
    x = s * s
    sens = np.exp(-x) * erfcx(s) / np.minimum(gammainc(1.5, x), gammainc(2.5, x))
    V = np.vander(u, deg + 1, increasing=True)
    w = sens / np.abs(y)
    c, *_ = np.linalg.lstsq(V * w[:, None], y * w, rcond=None)
    for _ in range(80):
        r = np.abs((V @ c - y) * w)
        w2 = w * np.sqrt(r / r.max()) + 1e-300
        c, *_ = np.linalg.lstsq(V * w2[:, None], y * w2, rcond=None)
    c32 = c.astype(np.float32)
    acc = np.full(u.shape, c32[-1], dtype=np.float32)
    u32 = u.astype(np.float32)
    for k in range(deg - 1, -1, -1):
        acc = (acc * u32 + c32[k]).astype(np.float32)
    e64 = np.abs((V @ c - y) * w).max()
    e32 = np.abs((acc.astype(np.float64) - y) * w).max()
    return c32, e64, e32


def fit_mp(f, w, a, b, deg, points=240, rounds=40):
    """Coefficients (lowest first) in t = (2 v - a - b) / (b - a) of the polynomial of degree deg whose error times w(v)
    is least on [a, b], as doubles, and that largest error with these."""
    # Chebyshev points: nearly minimax already before the reweighting
    t = [-mp.cos(mp.pi * (i + mp.mpf(1) / 2) / points) for i in range(points)]
    v = [(a + b + (b - a) * x) / 2 for x in t]
    y, sens = [f(x) for x in v], [w(x) for x in v]
    law = [mp.mpf(1)] * points
    best = None
    for _ in range(rounds):
        A = mp.matrix(points, deg + 1)
        r = mp.matrix(points, 1)
        for i in range(points):
            g = mp.sqrt(law[i]) * sens[i]
            for k in range(deg + 1):
                A[i, k] = g * mp.chebyt(k, t[i])
            r[i] = g * y[i]
        c = mp.lu_solve(A.T * A, A.T * r)
        e = [abs(mp.fsum(c[k] * mp.chebyt(k, t[i]) for k in range(deg + 1)) - y[i]) * sens[i] for i in range(points)]
        top = max(e)
        if best is None or top < best[0]:
            best = (top, c)
        law = [q * x / top for q, x in zip(law, e)]
        tot = mp.fsum(law)
        law = [q * points / tot + mp.mpf(10) ** -30 for q in law]
    # Chebyshev to power basis in t
    power = [mp.mpf(0)] * (deg + 1)
    T0, T1 = [mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]
    for k in range(deg + 1):
        T = T0 if k == 0 else T1
        for j, q in enumerate(T):
            power[j] += best[1][k] * q
        if k:
            T2 = [mp.mpf(0)] + [2 * q for q in T1]
            for j, q in enumerate(T0):
                T2[j] -= q
            T0, T1 = T1, T2
    return power


def as_doubles(c):
    return [float(q) for q in c]


def shift_to_origin(c, a, b):
    """The polynomial in v of one in t = (2 v - a - b) / (b - a)."""
    p, m = mp.mpf(2) / (b - a), -(a + b) / (b - a)
    out = [mp.mpf(0)]
    for q in reversed(c):
        nxt = [mp.mpf(0)] * (len(out) + 1)
        for j, r in enumerate(out):
            nxt[j] += r * m
            nxt[j + 1] += r * p
        nxt[0] += q
        out = nxt
    return out[:len(c)]


def horner(c, t):
    r = mp.mpf(0)
    for q in reversed(c):
        r = r * t + mp.mpf(q)
    return r


def m2_64(x):
    """sum_k x^k / Gamma(k + 7/2): P(5/2, x) = x^(5/2) e^-x times it."""
    return mp.hyp1f1(1, mp.mpf(7) / 2, x) / mp.gamma(mp.mpf(7) / 2)


def pe_64(u):
    s = 1 / u
    return s * mp.exp(s * s) * mp.erfc(s)


def gamma_p(a, x):
    return mp.gammainc(a, 0, x, regularized=True)


def float64_lines():
    mp.mp.dps = 40
    split, top = mp.mpf(3), mp.mpf(43)
    a, b = 1 / mp.sqrt(top), 1 / mp.sqrt(split)
    # a relative error r of P(3/2) or P(5/2) from one of Pe
    pe = as_doubles(fit_mp(pe_64, lambda u: u * mp.exp(-1 / u ** 2) / gamma_p(mp.mpf(5) / 2, 1 / u ** 2), a, b, 11))
    m2 = as_doubles(shift_to_origin(fit_mp(m2_64, lambda x: 1 / m2_64(x), mp.mpf(0), split, 15), mp.mpf(0), split))
    scale, shift = float(2 / (b - a)), float(-(a + b) / (b - a))
    e_pe = max(abs(horner(pe, mp.mpf(scale) * u + mp.mpf(shift)) - pe_64(u)) * u * mp.exp(-1 / u ** 2)
               / gamma_p(mp.mpf(5) / 2, 1 / u ** 2) for u in (a + (b - a) * i / 997 for i in range(998)))
    e_m2 = max(abs(horner(m2, x) / m2_64(x) - 1) for x in (split * i / 997 for i in range(998)))
    hi = float(mp.floor(mp.log(2) * 2 ** 40) / 2 ** 40)
    lo = float(mp.log(2) - mp.mpf(hi))
    num = lambda v: ", ".join("%.17e" % q for q in v)  # noqa: E731
    return [
        "/* Float64 form, x = s^2.  x < %d: sum_k x^k / Gamma(k + 7/2), relative error %s (of the" % (split, mp.nstr(e_m2, 2)),
        "   coefficients as doubles, in exact arithmetic). */",
        "static constexpr double VFMM64_M2_C[%d] = {%s};" % (len(m2), num(m2)),
        "/* %d <= x <= %d: s erfcx(s) in t = SCALE u + SHIFT, u = 1/s; relative error it causes in P(3/2, x) and" % (split, top),
        "   P(5/2, x): %s.  1 - P(5/2, %d) = %s. */" % (mp.nstr(e_pe, 2), top, mp.nstr(1 - gamma_p(mp.mpf(5) / 2, top), 2)),
        "static constexpr double VFMM64_PE_C[%d] = {%s};" % (len(pe), num(pe)),
        "#define VFMM64_PE_SCALE %.17e" % scale,
        "#define VFMM64_PE_SHIFT %.17e" % shift,
        "#define VFMM64_XSPLIT %.1f" % split,
        "#define VFMM64_XMAX %.1f" % top,
        "/* ln 2 = HI + LO, HI of 40 bits */",
        "#define VFMM64_LN2_HI %.17e" % hi,
        "#define VFMM64_LN2_LO %.17e" % lo,
    ]


def main():
    S_SPLIT = 1.0
    S_FIT_MAX = 6.3
    DEG_E = 5
    DEG_M = 5
    ce, e64, e32 = fit_cutoff(S_SPLIT, S_FIT_MAX, DEG_E)
    cm, m64, m32 = fit_rel(lambda x: hyp1f1(1.0, 3.5, x), 0.0, S_SPLIT ** 2, DEG_M)
    lines = [
        "/* Generated by gen_cutoff_fits.py -- do not edit. */",
        "#pragma once",
        "/* erfcx(s) ~= u * sum_k VFMM_ERFCX_C[k] u^k, u = 1/s, s in [%.1f, %.1f];" % (S_SPLIT, S_FIT_MAX),
        "   max error it causes in P(3/2, s^2), P(5/2, s^2), relative: %.2e (float64 coefs) /" % e64,
        "   %.2e (float32 Horner). */" % e32,
        "#define VFMM_ERFCX_DEG %d" % DEG_E,
        "static constexpr float VFMM_ERFCX_C[%d] = {%s};" % (DEG_E + 1, ", ".join("%.9ef" % v for v in ce)),
        "/* 1F1(1; 7/2; x) ~= sum_k VFMM_M2_C[k] x^k, x in [0, %.1f];" % (S_SPLIT ** 2),
        "   max rel. error %.2e (float64 coefs) / %.2e (float32 Horner). */" % (m64, m32),
        "#define VFMM_M2_DEG %d" % DEG_M,
        "static constexpr float VFMM_M2_C[%d] = {%s};" % (DEG_M + 1, ", ".join("%.9ef" % v for v in cm)),
        "/* branch point s = %.1f (x = s^2) between the two forms */" % S_SPLIT,
        "#define VFMM_CUTOFF_XSPLIT %.9ef" % (S_SPLIT ** 2),
    ] + float64_lines() + [""]
    with open(os.path.join(HERE, "cutoff_fits.h"), "w") as f:
        f.write("\n".join(lines))
    print("\n".join(lines))


if __name__ == "__main__":
    main()
