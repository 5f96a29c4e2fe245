"""Fit the binary32 polynomial cores of the mixed-precision transcendental
functions in exact.hip (atan_mixed, asinh_mixed, log_ratio_mixed).

Method: discrete minimax of the relative error by linear programming.  On a
dense grid of the reduced argument the coefficients c and a bound e solve
    minimise e  subject to  |sum_j c_j phi_j(x_k) - g(x_k)| <= e |f(x_k)|,
which is the Chebyshev (minimax) approximation on the grid; the LP is solved
with scipy's HiGHS.  The coefficients are then rounded to binary32 and the
whole core is evaluated as the device does (binary32 Horner with fused
multiply-adds, binary64 assembly) to report the achieved relative error of
the function itself.

  atan:  atan(s) = s + s^3 P(s^2) on |s| <= tan(pi/8) (the reduced range
         after the octant reduction), P of degree 5;
  atanh: 2 atanh(t) = 2 t + t^3 Q(t^2) on |t| <= 3 - 2 sqrt(2) (the range
         left by splitting off the binary exponent and folding the mantissa
         into [1/sqrt(2), sqrt(2)]), Q of degree 3; log and asinh use it.

The binary64 cores (atan2_64, log_ratio64) have the same forms with degrees
10 and 6: P and Q are interpolated at the Chebyshev points of the reduced
range in exact rational arithmetic (their Taylor series have rational
coefficients) and rounded once.

Run: python fit_cores.py   (prints the coefficients in the order Horner
evaluates them, highest degree first, and the achieved errors)."""
from __future__ import annotations

import math
from fractions import Fraction

import numpy as np
from scipy.optimize import linprog

TAN_PI_8 = np.tan(np.pi / 8)
ATANH_T = 3.0 - 2.0 * np.sqrt(2.0)


def minimax(z, target, weight, degree):
    """Coefficients a_0..a_degree of p(z) = sum a_j z^j minimising
    max_k |p(z_k) - target_k| / weight_k on the grid z."""
    # rows scaled so that the optimal residuals are of order one (the
    # solver's feasibility tolerance is absolute, about 1e-7)
    scale = 1e9
    A = np.vander(z, degree + 1, increasing=True) / weight[:, None] * scale
    b = target / weight * scale
    n = degree + 1
    # variables: a_0..a_degree, e; minimise e
    c = np.zeros(n + 1)
    c[-1] = 1.0
    A_ub = np.vstack([np.hstack([A, -np.ones((len(z), 1))]), np.hstack([-A, -np.ones((len(z), 1))])])
    b_ub = np.concatenate([b, -b])
    res = linprog(c, A_ub=A_ub, b_ub=b_ub, bounds=[(None, None)] * n + [(0, None)], method="highs")
    assert res.success, res.message
    return res.x[:n], res.x[-1] / scale


def fmaf(a, b, c):
    """binary32 fused multiply-add (the product of two binary32 numbers is
    exact in binary64; one rounding of the sum to binary32)."""
    return np.float32(np.float64(a) * np.float64(b) + np.float64(c))


def horner32(coef_hi_first, zf):
    p = np.float32(coef_hi_first[0]) * np.ones_like(zf)
    for c in coef_hi_first[1:]:
        p = fmaf(p, zf, np.float32(c))
    return p


def atan_core(P32, s):
    """s + s^3 P(s^2): s, z = s^2 and the assembly in binary64, P in binary32."""
    z = s * s
    P = horner32(P32, z.astype(np.float32)).astype(np.float64)
    return s + (s * z) * P


def atanh2_core(Q32, t):
    """2 atanh(t) = 2t + t^3 Q(t^2), Q in binary32."""
    t2 = t * t
    Q = horner32(Q32, t2.astype(np.float32)).astype(np.float64)
    return 2.0 * t + (t * t2) * Q


def fit_atan(degree=5, n=20000):
    s = np.linspace(1e-6, TAN_PI_8, n)
    z = s * s
    # (atan(s) - s) / s^3 = P(z); relative error of atan: s^3 |P - P*| / atan(s)
    target = (np.arctan(s) - s) / (s * z)
    weight = np.arctan(s) / (s * z)
    a, e = minimax(z, target, weight, degree)
    return a[::-1].astype(np.float32), e


def fit_atanh(degree=3, n=20000):
    t = np.linspace(1e-6, ATANH_T, n)
    t2 = t * t
    f = 2.0 * np.arctanh(t)
    target = (f - 2.0 * t) / (t * t2)
    weight = f / (t * t2)
    a, e = minimax(t2, target, weight, degree)
    return a[::-1].astype(np.float32), e


def achieved(P32, Q32, n=200001):
    s = np.linspace(-TAN_PI_8, TAN_PI_8, n)
    s = s[s != 0]
    ea = np.max(np.abs(atan_core(P32, s) - np.arctan(s)) / np.abs(np.arctan(s)))
    t = np.linspace(-ATANH_T, ATANH_T, n)
    t = t[t != 0]
    eh = np.max(np.abs(atanh2_core(Q32, t) - 2.0 * np.arctanh(t)) / np.abs(2.0 * np.arctanh(t)))
    return ea, eh


def interpolate64(taylor, b, degree, terms=60):
    """(coefficients highest degree first, largest error) of the polynomial
    through g(z) = sum_k taylor(k) z^k at the Chebyshev points of [0, b]."""
    n = degree + 1
    x = [Fraction(b) * Fraction((1.0 + math.cos(math.pi * (2 * i + 1) / (2 * n))) / 2.0) for i in range(n)]

    def g(z):
        return sum(taylor(k) * z ** k for k in range(terms))

    c = [g(z) for z in x]
    for j in range(1, n):  # divided differences
        for i in range(n - 1, j - 1, -1):
            c[i] = (c[i] - c[i - 1]) / (x[i] - x[i - j])
    poly = [Fraction(0)]
    for i in range(n - 1, -1, -1):  # Newton's form to powers of z
        poly = [(poly[k - 1] if k else 0) - x[i] * (poly[k] if k < len(poly) else 0) for k in range(len(poly) + 1)]
        poly[0] += c[i]
    poly = poly[:n]
    grid = [Fraction(b) * k / 200 for k in range(201)]
    err = max(abs(sum(a * z ** k for k, a in enumerate(poly)) - g(z)) for z in grid)
    return [float(a) for a in poly[::-1]], float(err)


def fit_atan64(degree=10):
    return interpolate64(lambda k: Fraction((-1) ** (k + 1), 2 * k + 3), math.tan(math.pi / 8) ** 2, degree)


def fit_atanh64(degree=6):
    return interpolate64(lambda k: Fraction(2, 2 * k + 3), (3.0 - 2.0 * math.sqrt(2.0)) ** 2, degree)


if __name__ == "__main__":
    P, e1 = fit_atan()
    Q, e2 = fit_atanh()
    print("atan  P (highest degree first):", ", ".join(f"{float(c)!r}f" for c in P), f"  (LP bound {e1:.2e})")
    print("atanh Q (highest degree first):", ", ".join(f"{float(c)!r}f" for c in Q), f"  (LP bound {e2:.2e})")
    ea, eh = achieved(P, Q)
    print(f"achieved relative error with binary32 coefficients: atan {ea:.2e}, 2 atanh {eh:.2e}")
    for name, (C, e) in (("atan", fit_atan64()), ("atanh", fit_atanh64())):
        print(f"binary64 {name} (highest degree first):", ", ".join(repr(c) for c in C), f"  (within {e:.1e})")
