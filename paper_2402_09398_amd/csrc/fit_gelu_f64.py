"""Derives the constants of gelu_f64() and exp_parts_f64() in lessdec_common.h.

Upper tail of the standard normal, t >= 0: Q(t) = exp(-t^2 / 2) u q(u) with u = 1 / (1 + p t).  exp(t^2/2) Q(t) is smooth and slowly
decaying, so that a polynomial q of degree 16, interpolated at the Chebyshev points of u over 0 <= t <= 8 and written about
a point in the middle (which keeps the coefficients near 1 and their rounding small), takes t Q(t) to 1.1e-17 with the
coefficients rounded to fp64.  All in 50 digits; beyond t = 8 t Q(t) is below 1e-14 and decays faster than q errs.

e^r for |r| <= ln 2 / 2: 1 + r + r^2/2 + r^3 p(r), p of degree 8, interpolated at the Chebyshev points.
"""
import math
from decimal import Decimal, getcontext

getcontext().prec = 50
P, N, CENTRE, TOP = Decimal("0.2"), 16, Decimal("0.6875"), Decimal(8)
PI = Decimal("3.14159265358979323846264338327950288419716939937510582097494459")


def scaled_tail(t):
    """exp(t^2 / 2) Q(t): the series of the normal's distribution below 4, its continued fraction above."""
    t = Decimal(t)
    if t < 4:
        s, term, k = Decimal(0), t, 0
        while abs(term) > Decimal(10) ** -48:
            s += term
            k += 1
            term = term * t * t / (2 * k + 1)
        return (t * t / 2).exp() / 2 - s / (2 * PI).sqrt()
    f = Decimal(0)
    for k in range(400, 0, -1):
        f = Decimal(k) / (t + f)
    return 1 / ((t + f) * (2 * PI).sqrt())


def fit():
    """Coefficients of q about CENTRE, lowest first, as Decimals."""
    low = 1 / (1 + P * TOP)
    half, mid = (1 - low) / 2, (1 + low) / 2
    us = [half * Decimal(math.cos(math.pi * (2 * i + 1) / (2 * N + 2))) + mid for i in range(N + 1)]
    c = [scaled_tail((1 / u - 1) / P) / u for u in us]
    for j in range(1, N + 1):                               # divided differences
        for i in range(N, j - 1, -1):
            c[i] = (c[i] - c[i - 1]) / (us[i] - us[i - j])
    poly = [c[N]]
    for i in range(N - 1, -1, -1):                          # Newton's form to powers of w = u - CENTRE
        root = us[i] - CENTRE
        grown = [Decimal(0)] * (len(poly) + 1)
        for k, v in enumerate(poly):
            grown[k + 1] += v
            grown[k] -= v * root
        grown[0] += c[i]
        poly = grown
    return poly


def tail(t, coefficients):
    """t Q(t) from the polynomial, exactly, and the true value."""
    t = Decimal(t)
    u = 1 / (1 + P * t)
    q = Decimal(0)
    for v in reversed(coefficients):
        q = q * (u - CENTRE) + Decimal(v)
    e = (-t * t / 2).exp()
    return t * u * q * e, t * scaled_tail(t) * e


def fit_exp(degree=11, known=3):
    """Coefficients of r^0 .. r^degree, as floats; the first `known` are those of the series."""
    half, n = Decimal(2).ln() / 2 * Decimal("1.0001"), degree - known + 1
    rs = [half * Decimal(math.cos(math.pi * (2 * i + 1) / (2 * n))) for i in range(n)]
    c = [sum(r ** k / math.factorial(k + known) for k in range(40)) for r in rs]
    for j in range(1, n):                                   # divided differences
        for i in range(n - 1, j - 1, -1):
            c[i] = (c[i] - c[i - 1]) / (rs[i] - rs[i - j])
    poly = [c[-1]]
    for i in range(n - 2, -1, -1):                          # Newton's form to powers
        poly = [c[i] - poly[0] * rs[i]] + [poly[k] - poly[k + 1] * rs[i] for k in range(len(poly) - 1)] + [poly[-1]]
    return [1 / math.factorial(k) for k in range(known)] + [float(v) for v in poly]


def exp_error(r, coefficients):
    """Relative error of e^r from these coefficients, exactly evaluated."""
    r, p = Decimal(r), Decimal(0)
    for v in reversed(coefficients):
        p = p * r + Decimal(v)
    return float(p / r.exp() - 1)


if __name__ == "__main__":
    rounded = [float(v) for v in fit()]
    for k, v in enumerate(rounded):
        print(f"q{k} = {v:.17e}")
    print("t Q(t) within", max(abs(float(a - b)) for a, b in (tail(0.03 * i, rounded) for i in range(300))))
    for k, v in enumerate(fit_exp()):
        print(f"e{k} = {v:.17e}")
    print("e^r within", max(abs(exp_error(0.34658 * i / 100, fit_exp())) for i in range(-100, 101)))
