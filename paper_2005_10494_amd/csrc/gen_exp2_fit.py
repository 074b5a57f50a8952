"""Writes exp2_fit.hpp: the coefficients of the double-precision 2^f on
|f| <= 1/2 that the FP64 integrands evaluate after splitting an exponent into
its nearest integer and the rest.

Form.  2^f = 1 + f Q(f), Q(f) = (2^f - 1)/f interpolated at the Chebyshev nodes
of [-1/2, 1/2] in 40-digit arithmetic, so 2^0 is exactly 1 and the error stays
within a small factor of the minimax one.  DEG is the degree of the whole
polynomial.  Degree 11 leaves 2e-17 relative, below the rounding of the evaluation
(1.1e-16); degree 10 would leave 5.7e-16.

The script replays the device's evaluation (Horner with fused multiply-adds)
against 40-digit values and records the errors in the header.

Run: python paper_2005_10494_amd/csrc/gen_exp2_fit.py
"""
import os

import mpmath as mp

DEG = 11
HERE = os.path.dirname(os.path.abspath(__file__))


def fit(deg=DEG):
    """Coefficients c_0 = 1, c_1 .. c_deg, rounded to double."""
    mp.mp.dps = 40
    n = deg   # Q has degree deg - 1
    x = [mp.cos(mp.pi * (2 * i + 1) / (2 * n)) / 2 for i in range(n)]
    A = mp.matrix(n, n)
    b = mp.matrix(n, 1)
    for i in range(n):
        b[i] = mp.expm1(x[i] * mp.log(2)) / x[i] if x[i] != 0 else mp.log(2)
        for j in range(n):
            A[i, j] = x[i] ** j
    q = mp.lu_solve(A, b)
    return [1.0] + [float(q[i]) for i in range(n)]


def replay(c, f):
    """Horner in double precision, each fused multiply-add rounded once."""
    p = c[-1]
    for a in reversed(c[:-1]):
        p = float(mp.mpf(p) * mp.mpf(f) + mp.mpf(a))
    return p


def errors(c, n=4001):
    """Largest relative error: of the polynomial, and of its evaluation."""
    mp.mp.dps = 40
    poly = evald = mp.mpf(0)
    for i in range(n):
        f = -0.5 + i / (n - 1)
        ref = mp.mpf(2) ** mp.mpf(f)
        exact = mp.polyval([mp.mpf(a) for a in reversed(c)], mp.mpf(f))
        poly = max(poly, abs(exact / ref - 1))
        evald = max(evald, abs(mp.mpf(replay(c, f)) / ref - 1))
    return float(poly), float(evald)


def main():
    c = fit()
    poly, evald = errors(c)
    with open(os.path.join(HERE, "exp2_fit.hpp"), "w") as f:
        f.write("// Generated by gen_exp2_fit.py; do not edit.\n")
        f.write("// 2^f = sum_(i=0..%d) c_i f^i on |f| <= 1/2, c_0 first; against 40-digit values the\n" % DEG)
        f.write("// polynomial is within %.2e relative, its double-precision evaluation within %.2e.\n" % (poly, evald))
        f.write("#pragma once\n\nnamespace bmd {\nconstexpr int kExp2Deg = %d;\n" % DEG)
        f.write("constexpr double kExp2Fit[kExp2Deg + 1] = {\n")
        for a in c:
            f.write("    %s,  // %.17g\n" % (float(a).hex(), a))
        f.write("};\n}  // namespace bmd\n")


if __name__ == "__main__":
    main()
