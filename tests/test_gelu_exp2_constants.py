"""gelu_exp2_f32 of csrc/lessdec_common.h, the activation of the feature maps' hidden layers (Sec. 3.2 names GELU): its constants are
the ones csrc/fit_gelu_poly.py derives, and evaluated as the kernels evaluate it it is no further from x Phi(x) than
gelu_fast_f32."""
import re

import numpy as np
from scipy.special import erfc

from tests.test_gelu_constants import CSRC, _fit_module, _header_constants


def _constants():
    src = (CSRC / "lessdec_common.h").read_text()
    body = src[src.index("float gelu_exp2_f32"):]
    body = body[:body.index("\n}\n")]
    first = float(re.search(r"float p = (-?\d\.\d+e[-+]\d+)f;", body).group(1))
    rest = [float(x) for x in re.findall(r"p = fmaf\(p, t, (-?\d\.\d+(?:e[-+]\d+)?)f\);", body)]
    return ([first] + rest)[::-1]                  # c0 .. c8


def test_constants_are_the_fitted_ones():
    c, worst = _fit_module().fit_log2()
    got = _constants()
    assert len(got) == 9 and got[0] == -1.0 and got[-1] < 0
    # the fit's digits depend a little on the linear algebra library; what they may change is the error of t Q(t)
    t = np.linspace(0, 7, 7001)
    q = np.exp2(np.polynomial.polynomial.polyval(t, got))
    assert worst < 1.2e-8 and np.abs(t * q - t * 0.5 * erfc(t / np.sqrt(2))).max() < 1.1 * worst
    np.testing.assert_allclose(got, c, rtol=2e-2)


def test_error_against_the_other_form():
    fit = _fit_module()
    p, horner = _header_constants("gelu_fast_f32")
    x = np.concatenate([np.linspace(-12, 12, 400001), np.geomspace(1e-6, 1, 2001)])
    exact = 0.5 * x.astype(np.float32).astype(np.float64) * erfc(-x.astype(np.float32).astype(np.float64) / np.sqrt(2))
    new = np.abs(fit.gelu_exp2_32(x, _constants()).astype(np.float64) - exact)
    old = np.abs(fit.gelu32(x, p, np.array(horner[::-1])).astype(np.float64) - exact)
    for lo, hi in ((0, 1e-3), (1e-3, 0.1), (0.1, 0.5), (0.5, 2), (2, 4), (4, 13)):
        k = (np.abs(x) >= lo) & (np.abs(x) < hi)
        # root mean square: no larger; largest: half a unit in the last place of x and the approximation's own
        assert np.sqrt((new[k] ** 2).mean()) <= 1.02 * np.sqrt((old[k] ** 2).mean()) + 1e-10
        assert (new[k] <= 6e-8 * np.abs(x[k]) + 3e-8).all()


def test_far_out():
    x = np.array([20.0, 1e3, 1e6, 6e9, 1e12], np.float32)
    with np.errstate(over="ignore"):
        got = _fit_module().gelu_exp2_32(np.concatenate([x, -x]), _constants())
    np.testing.assert_array_equal(got, np.concatenate([x, np.zeros_like(x)]))
