"""gelu_exp2_f32 of csrc/lessdec_common.h, the activation of the feature maps' hidden layers (Sec. 3.2 names GELU): its constants are
the ones csrc/fit_gelu_poly.py derives, and on either side of zero it is no further from x Phi(x) than the form with a reciprocal."""
import numpy as np
import pytest
from scipy.special import erfc

from tests.header_on_host import body, horner, on_host
from tests.test_gelu_constants import _fit_module


@pytest.fixture(scope="module")
def gelu():
    return on_host("gelu_exp2_f32")["gelu_exp2_f32"]


def exact(x):
    x = x.astype(np.float64)
    return 0.5 * x * erfc(-x / np.sqrt(2))


def test_constants_are_the_fitted_ones():
    fit = _fit_module()
    c, _ = fit.fit_log2()
    text = body("gelu_exp2_f32")
    got = horner(text, "p", "s")[::-1]
    assert len(got) == 11 and got[-1] < 0 and f"s = t - {fit.CENTRE}f" in text
    # the fit's digits depend a little on the linear algebra library; the error is the other test's
    np.testing.assert_allclose(got, c, rtol=0.1, atol=1e-6)


# Half units on either side of zero.  Below -6.5 gelu is above -2.7e-10: the error's size alone counts there.
RANGES = [(a / 2, (a + 1) / 2) for a in range(-13, 13)] + [(6.5, 13.0), (-0.1, -0.01), (0.01, 0.1), (-0.01, 0.01)]


@pytest.mark.parametrize("lo,hi", RANGES, ids=lambda v: str(v))
def test_no_further_off_than_the_form_with_a_reciprocal(gelu, lo, hi):
    fit = _fit_module()
    x = np.random.default_rng(5).uniform(lo, hi, 40001).astype(np.float32)
    rms = lambda y: np.sqrt(((y.astype(np.float64) - exact(x)) ** 2).mean())  # noqa: E731
    # 40001 samples give a root mean square to 1 % (their squares vary by about twice their mean)
    assert rms(gelu(x)) <= 1.01 * rms(fit.gelu32(x, fit.P, fit.fit()))


def test_far_below_zero(gelu):
    x = -np.linspace(6.5, 40, 40001).astype(np.float32)
    assert np.abs(gelu(x) - exact(x)).max() < 3e-13


def test_far_out(gelu):
    x = np.geomspace(7, 3e38, 4001).astype(np.float32)
    np.testing.assert_array_equal(gelu(x), x)                       # t Q(t) is below half a unit in the last place
    assert np.abs(gelu(-x)).max() < 1e-11 and (gelu(-x[x > 15]) == 0).all()
    assert np.isnan(gelu(np.array([np.nan, -np.inf], np.float32))).all()
