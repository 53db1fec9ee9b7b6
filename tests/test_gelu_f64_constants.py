"""gelu_f64 of csrc/lessdec_common.h, the activation of the fp64 feature maps (Sec. 3.2 names GELU): its constants are the ones
csrc/fit_gelu_f64.py derives, and evaluated in fp64 it stays within a unit in the last place of max(|x|, 1/4) of x Phi(x)."""
import importlib.util
import math
import re
from decimal import Decimal

import numpy as np

from tests.test_gelu_constants import CSRC


def _fit():
    spec = importlib.util.spec_from_file_location("fit_gelu_f64", CSRC / "fit_gelu_f64.py")
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _body():
    src = (CSRC / "lessdec_common.h").read_text()
    body = src[src.index("double gelu_f64(double x)"):]
    return body[:body.index("\n}\n")]


def _horner(name, arg):
    body = _body()
    first = float(re.search(rf"double {name} = (-?[\d.]+e[-+]\d+);", body).group(1))
    return [first] + [float(v) for v in re.findall(rf"{name} = fma\({name}, {arg}, (-?[\d.]+(?:e[-+]\d+)?)\);", body)]


def test_constants():
    fit = _fit()
    q = _horner("a", "w")[::-1]
    assert len(q) == fit.N + 1 and all(abs(a - float(b)) <= 1e-15 * abs(a) for a, b in zip(q, fit.fit()))
    assert max(abs(float(a - b)) for a, b in (fit.tail(0.05 * i, q) for i in range(180))) < 2e-17
    assert f"fma({fit.P}, t, 1.0)" in _body() and f"u - {fit.CENTRE};" in _body()
    e = _horner("e", "r")[::-1]
    assert len(e) == 13 and all(abs(v * math.factorial(k) - 1) < 1e-15 for k, v in enumerate(e))


def test_evaluation_error():
    fit = _fit()
    wide = np.longdouble

    def fma(a, b, c):
        return np.float64(wide(a) * wide(b) + wide(c))

    q, p = _horner("a", "w"), _horner("e", "r")
    for x in np.concatenate([np.linspace(-9, 9, 361), [1e-3, -1e-3, 0.0]]):
        t = np.float64(abs(x))
        u = np.float64(1) / fma(0.2, t, 1.0)
        a, w = q[0], u - 0.6875
        for v in q[1:]:
            a = fma(a, w, v)
        s = -0.5 * t * t
        n = np.rint(s * 1.44269504088896338700e+00)
        r = fma(n, -1.90821492927058770002e-10, fma(n, -6.93147180369123816490e-01, s))
        e = p[0]
        for v in p[1:]:
            e = fma(e, r, v)
        tq = t * (a * u * np.ldexp(e, int(n)))
        got = x - tq if x >= 0 else -tq
        true = fit.tail(float(t), [0.0])[1] if t > 0 else Decimal(0)
        want = Decimal(float(x)) - true if x >= 0 else -true
        assert abs(float(Decimal(float(got)) - want)) <= 2.3e-16 * max(abs(x), 0.25), x
