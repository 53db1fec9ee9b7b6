"""Derives the constants of exp2_f64() in lessdec_digits.h.

2^y = 2^n 2^f with n the integer nearest to y and |f| <= 1/2.  2^f is taken as the polynomial of degree 9
through its values at the ten Chebyshev points of [-1/2, 1/2]; the error of such an interpolation is at
most (ln 2)^10 sqrt(2) / (10! 2^9 4^10) = 1.8e-14 times the largest factor of the remainder.  Computed in
exact fractions from values of 30 digits, so that only the printing rounds.  Prints c_0 .. c_9 and the largest
relative error of a float64 evaluation by Horner's rule.
"""
from fractions import Fraction

import numpy as np

DEGREE = 9


def _exp2(x):
    """2^x for a Fraction |x| <= 1/2, its Taylor series to far below 1e-30."""
    ln2 = sum((Fraction(1, k * 2 ** k) for k in range(1, 120)), Fraction(0))
    term = total = Fraction(1)
    for k in range(1, 40):
        term = (term * ln2 * x / k).limit_denominator(10 ** 45)
        total += term
    return total


def fit(degree=DEGREE):
    n = degree + 1
    xs = [Fraction(float(np.cos(np.pi * (2 * i + 1) / (2 * n)) / 2)) for i in range(n)]
    ys = [_exp2(x) for x in xs]
    for k in range(1, n):                               # divided differences
        for i in range(n - 1, k - 1, -1):
            ys[i] = (ys[i] - ys[i - 1]) / (xs[i] - xs[i - k])
    c = [Fraction(0)] * n                               # Newton's form to powers
    for k in range(n - 1, -1, -1):
        c = [(c[i - 1] if i else Fraction(0)) - xs[k] * c[i] for i in range(n)]
        c[0] += ys[k]
    return [float(x) for x in c]


def evaluate(c, f):
    p = np.full_like(f, c[-1])
    for x in c[-2::-1]:
        p = p * f + x
    return p


if __name__ == "__main__":
    c = fit()
    for k, v in enumerate(c):
        print(f"c{k} = {v!r}")
    f = np.linspace(-0.5, 0.5, 200001)
    print("largest relative error on [-1/2, 1/2]:", np.abs(evaluate(c, f) / np.exp2(f.astype(np.longdouble)) - 1).max())
