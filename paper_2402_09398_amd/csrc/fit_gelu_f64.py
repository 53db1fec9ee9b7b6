"""Derives the constants of gelu_f64() and exp_parts_f64() in lessdec_common.h.

Upper tail of the standard normal, t >= 0: Q(t) = exp(-t^2 / 2) F(t), F(t) = 1/2 + c_1 v + ... + c_N v^N with
v = t / (1 + p t).  F decays smoothly from 1/2 to 1 / (t sqrt(2 pi)), and small t have small v, so that neither the
polynomial nor the division costs digits there.  Weighted least squares over 0 <= t <= 39, beyond which Q is below the smallest fp64
number, in the relative error of F; the weight allows (1 + 0.6 t^2) 1e-17, a tenth of what rounding -t^2 / 2 to fp64 costs.  The
coefficients are rounded to fp64 one after the other, lowest first, and the others fitted again.  All in 90 digits.

e^r for |r| <= ln 2 / 2: 1 + r + r^2/2 + r^3 p(r), p of degree 8, interpolated at the Chebyshev points.
"""
import math
from decimal import Decimal, getcontext

getcontext().prec = 90
P, N, TOP = Decimal("0.2"), 20, 39
PI = Decimal("3.14159265358979323846264338327950288419716939937510582097494459230781640628620899862803482534211706798")


def scaled_tail(t):
    """F(t) = exp(t^2 / 2) Q(t): the series of the normal's distribution below 4, its continued fraction above."""
    t = Decimal(t)
    if t < 4:
        s, term, k = Decimal(0), t, 0
        while abs(term) > Decimal(10) ** -80:
            s += term
            k += 1
            term = term * t * t / (2 * k + 1)
        return (t * t / 2).exp() / 2 - s / (2 * PI).sqrt()
    f = Decimal(0)
    for k in range(600, 0, -1):
        f = Decimal(k) / (t + f)
    return 1 / ((t + f) * (2 * PI).sqrt())


def _solve(a, b):
    n = len(b)
    for i in range(n):
        for j in range(i + 1, n):
            m = a[j][i] / a[i][i]
            for k in range(i, n):
                a[j][k] -= m * a[i][k]
            b[j] -= m * b[i]
    for i in reversed(range(n)):
        b[i] = (b[i] - sum(a[i][k] * b[k] for k in range(i + 1, n))) / a[i][i]
    return b


def fit(points=120):
    """c_1 .. c_N as floats."""
    low = 1 / (1 + P * TOP)
    us = [(1 + low) / 2 + (1 - low) / 2 * Decimal(math.cos(math.pi * (2 * i + 1) / (2 * points))) for i in range(points)]
    ts = [(1 / u - 1) / P for u in us]
    vs = [t * u for t, u in zip(ts, us)]
    fs = [scaled_tail(t) for t in ts]
    w2 = [1 / (f * (1 + Decimal("0.6") * t * t)) ** 2 for f, t in zip(fs, ts)]
    powers = [[v ** k for k in range(N + 1)] for v in vs]
    moments = [sum(w * row[1] ** k for w, row in zip(w2, powers)) for k in range(2 * N + 1)]
    known = [Decimal("0.5")]
    while len(known) <= N:
        free = range(len(known), N + 1)
        rest = [f - sum(c * x for c, x in zip(known, row)) for f, row in zip(fs, powers)]
        b = [sum(w * r * row[j] for w, r, row in zip(w2, rest, powers)) for j in free]
        known.append(Decimal(float(_solve([[moments[j + k] for k in free] for j in free], b)[0])))
    return [float(c) for c in known[1:]]


def error(t, coefficients):
    """Relative error of F at t from these coefficients, exactly evaluated."""
    t = Decimal(t)
    v = t / (1 + P * t)
    q = Decimal(0)
    for c in reversed(coefficients):
        q = (q + Decimal(c)) * v
    f = scaled_tail(t)
    return float((q + Decimal("0.5") - f) / f)


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
    c = fit()
    for k, value in enumerate(c, 1):
        print(f"c{k} = {value:.17e}")
    print("of the allowed error", max(abs(error(0.0154 * i * i, c)) / (1e-17 * (1 + 0.6 * (0.0154 * i * i) ** 2)) for i in range(1, 50)))
    for k, v in enumerate(fit_exp()):
        print(f"e{k} = {v:.17e}")
    print("e^r within", max(abs(exp_error(0.34658 * i / 100, fit_exp())) for i in range(-100, 101)))
