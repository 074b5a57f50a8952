"""Writes mills_fit.hpp: the coefficients of Mills' ratio M(y) = (1 - Phi(y))/phi(y),
y >= 0, that the FP64 derivatives evaluate (a density times a normal probability
in its lower tail is a density times a Mills ratio).

Form.  With r = 1/(y + K) and s = 1 - 2 K r in [-1, 1), M = r F(s), and
F(s) = (y + K) M(y) is smooth on [-1, 1] (F(1) = 1): interpolated at the
Chebyshev nodes in 40-digit arithmetic and written in powers of s.  K = 4 and
degree 24 leave 1e-16 relative; K from 2 to 5 need 24 to 28 for it.

The script replays the device's evaluation (Horner with fused multiply-adds)
against 40-digit values and records the errors in the header.

Run: python paper_2005_10494_amd/csrc/gen_mills_fit.py
"""
import os

import mpmath as mp

K, DEG = 4, 24
HERE = os.path.dirname(os.path.abspath(__file__))


def mills(y):
    """M(y) in the working precision (the continued fraction beyond y = 60)."""
    if y < 60:
        return mp.erfc(y / mp.sqrt(2)) * mp.exp(y * y / 2) * mp.sqrt(mp.pi / 2)
    t = y
    for k in range(30, 0, -1):
        t = y + k / t
    return 1 / t


def fit():
    """Coefficients c_0 .. c_DEG of F in powers of s, rounded to double."""
    mp.mp.dps = 40
    n = DEG + 1
    th = [mp.pi * (2 * i + 1) / (2 * n) for i in range(n)]
    f = []
    for t in th:
        y = K * (1 + mp.cos(t)) / (1 - mp.cos(t))
        f.append((y + K) * mills(y))
    cheb = [(1 if k == 0 else 2) * mp.fsum(f[i] * mp.cos(k * th[i]) for i in range(n)) / n for k in range(n)]
    out = [mp.mpf(0)] * n
    t0, t1 = [mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]   # T_0, T_1 in powers of s
    for c in cheb:
        for i, a in enumerate(t0):
            out[i] += c * a
        t2 = [mp.mpf(0)] + [2 * a for a in t1]
        for i, a in enumerate(t0):
            t2[i] -= a
        t0, t1 = t1, t2
    return [float(a) for a in out]


def _fma(a, b, c):
    return float(mp.mpf(a) * mp.mpf(b) + mp.mpf(c))


def replay(c, y):
    """The device's evaluation in double precision, the reciprocal rounded once."""
    r = float(1 / (mp.mpf(y) + K))
    s = _fma(-2.0 * K, r, 1.0)
    p = c[-1]
    for a in reversed(c[:-1]):
        p = _fma(p, s, a)
    return r * p


def errors(c, n=1500):
    """Largest relative error: of the fit, and of its evaluation."""
    mp.mp.dps = 40
    poly = evald = mp.mpf(0)
    for i in range(n):
        y = 40.0 * (i / (n - 1)) ** 2
        ref = mills(mp.mpf(y))
        r = 1 / (mp.mpf(y) + K)
        p = mp.polyval([mp.mpf(a) for a in reversed(c)], 1 - 2 * K * r) * r
        poly = max(poly, abs(p / ref - 1))
        evald = max(evald, abs(mp.mpf(replay(c, y)) / ref - 1))
    return float(poly), float(evald)


def main():
    c = fit()
    poly, evald = errors(c)
    with open(os.path.join(HERE, "mills_fit.hpp"), "w") as f:
        f.write("// Generated by gen_mills_fit.py; do not edit.\n")
        f.write("// (y + K) M(y) = sum_(i=0..%d) c_i s^i, s = 1 - 2 K / (y + K), M Mills' ratio of the normal, y >= 0;\n" % DEG)
        f.write("// against 40-digit values the polynomial is within %.2e relative, its evaluation within %.2e.\n" % (poly, evald))
        f.write("#pragma once\n\nnamespace bmd {\nconstexpr double kMillsK = %d;\nconstexpr int kMillsDeg = %d;\n" % (K, DEG))
        f.write("constexpr double kMillsFit[kMillsDeg + 1] = {\n")
        for a in c:
            f.write("    %s,  // %.17g\n" % (float(a).hex(), a))
        f.write("};\n}  // namespace bmd\n")


if __name__ == "__main__":
    main()
