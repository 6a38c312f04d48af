"""Generate split_poly64.h: the polynomials behind the FP64 short-range factor.

The short-range factor of the PM split (sec. 3.1, Eq. equ:split) is
    g(x) = erfc(x) + (2x/sqrt(pi)) exp(-x^2) = exp(-x^2) P(x),
    P(x) = exp(x^2) erfc(x) + 2x/sqrt(pi),
with P smooth and between 1 and 2.8 on [0, X_MAX]: the product keeps its
relative precision up to the cut, where g is 0.017 (1 - x^3 H(x^2), the form
of the FP32 path, loses a factor of 60 there).  P is its Chebyshev series on
[0, X_MAX] in powers of t = 2x/X_MAX - 1; exp(-x^2) = 2^-n 2^-f with n the
integer nearest to x^2 log2(e), and 2^-f its Chebyshev series on [-1/2, 1/2]
in powers of f.  Coefficients and nodes at 60 digits.

    python gen_split_poly64.py [out.h]         # default: rewrites split_poly64.h beside it
"""
import os
import sys

import mpmath as mp
import numpy as np

X_MAX = 2.26            # as in gen_split_poly.py
DEGREE_P, DEGREE_E = 23, 11
NODES = 80


def P(x):
    return mp.exp(x * x) * mp.erfc(x) + 2 * x / mp.sqrt(mp.pi)


def series(f, lo, hi, degree, scale):
    """Power coefficients, in the variable s scale with s in [-1, 1], of the
    Chebyshev series of f on [lo, hi] cut at `degree`."""
    mp.mp.dps = 60
    th = [mp.pi * (k + mp.mpf(1) / 2) / NODES for k in range(NODES)]
    v = [f((hi + lo) / 2 + (hi - lo) / 2 * mp.cos(a)) for a in th]
    cheb = [2 * sum(vk * mp.cos(j * a) for vk, a in zip(v, th)) / NODES for j in range(degree + 1)]
    cheb[0] /= 2
    power = [mp.mpf(0)] * (degree + 1)
    t0, t1 = [mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]
    for j in range(degree + 1):
        for i, c in enumerate(t0):
            power[i] += cheb[j] * c
        t2 = [mp.mpf(0)] + [2 * c for c in t1]
        for i, c in enumerate(t0):
            t2[i] -= c
        t0, t1 = t1, t2
    return [float(c / mp.mpf(scale) ** i) for i, c in enumerate(power)]


def check(f, c, lo, hi, var):
    """Max relative error of the rounded coefficients, in exact arithmetic."""
    mp.mp.dps = 40
    worst = mp.mpf(0)
    for x in np.linspace(float(lo), float(hi), 1501):
        x = mp.mpf(float(x))
        p = sum(mp.mpf(ci) * var(x) ** i for i, ci in enumerate(c))
        worst = max(worst, abs(p / f(x) - 1))
    return float(worst)


def main():
    here = os.path.dirname(os.path.abspath(__file__))
    out = sys.argv[1] if len(sys.argv) > 1 else os.path.join(here, "split_poly64.h")
    xm, half = mp.mpf(X_MAX), mp.mpf(1) / 2
    two = lambda f: mp.mpf(2) ** -f
    cp = series(P, mp.mpf(0), xm, DEGREE_P, 1)
    ce = series(two, -half, half, DEGREE_E, half)
    ep = check(P, cp, 0, xm, lambda x: 2 * x / xm - 1)
    ee = check(two, ce, -half, half, lambda f: f)
    with open(out, "w") as f:
        f.write("// Generated by gen_split_poly64.py -- do not edit.\n")
        f.write("// g(x) = exp(-x^2) P(x).  P(x) = sum_j SPLIT64_P[j] t^j, t = 2x/SPLIT64_X_MAX - 1, x in\n")
        f.write("// [0, SPLIT64_X_MAX]; 2^-f = sum_j SPLIT64_E[j] f^j, f in [-1/2, 1/2].  Checked max relative\n")
        f.write("// errors of the rounded coefficients (exact arithmetic): %.2e and %.2e.\n" % (ep, ee))
        f.write("#pragma once\n")
        f.write("#define SPLIT64_X_MAX %.17g\n" % X_MAX)
        for name, c in (("P", cp), ("E", ce)):
            f.write("#define SPLIT64_DEGREE_%s %d\n" % (name, len(c) - 1))
            f.write("static constexpr double SPLIT64_%s[%d] = {\n" % (name, len(c)))
            for ci in c:
                f.write("    %.17e,\n" % ci)
            f.write("};\n")
    print("P degree %d: %.2e; 2^-f degree %d: %.2e" % (DEGREE_P, ep, DEGREE_E, ee))


if __name__ == "__main__":
    main()
