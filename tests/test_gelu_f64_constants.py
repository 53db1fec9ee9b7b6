"""gelu_f64 of csrc/lessdec_common.h, the activation of the fp64 feature maps (Sec. 3.2 names GELU): its constants are the ones
csrc/fit_gelu_f64.py derives, and in every range, on either side of zero and far below it, it is no further from x Phi(x) than
0.5 x erfc(-x / sqrt 2) in fp64."""
import importlib.util
from decimal import Decimal

import numpy as np
import pytest
from scipy.special import erfc

from tests.header_on_host import CSRC, body, horner, on_host


@pytest.fixture(scope="module")
def fit():
    spec = importlib.util.spec_from_file_location("fit_gelu_f64", CSRC / "fit_gelu_f64.py")
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.fixture(scope="module")
def gelu():
    return on_host("gelu_f64")["gelu_f64"]


def test_constants(fit):
    c = horner(body("gelu_f64"), "a", "v")[::-1]
    assert len(c) == fit.N + 1 and c[0] == 0.5 and f"fma({fit.P}, t, 1.0)" in body("gelu_f64")
    # the points of the fit are cosines of a math library: its digits beyond those that matter may differ
    np.testing.assert_allclose(c[1:6], fit.fit()[:5], rtol=1e-6, atol=0)
    assert max(abs(fit.error(0.0154 * i * i, c[1:])) / (1e-17 * (1 + 0.6 * (0.0154 * i * i) ** 2)) for i in range(1, 50)) < 2


# Relative error.  numpy's erfc is nearly correctly rounded about zero, closer than the math library's on the GPU (1.0e-16 on
# [1/10, 1/2], 1.1e-16 on [-1/2, -1/10]): there the bound is that one's root mean square, elsewhere the form in fp64 here.
RANGES = [(-36, -20, None), (-20, -9, None), (-9, -5, None), (-5, -3, None), (-3, -2, None), (-2, -1, None), (-1, -0.5, 1.37e-16),
          (-0.5, -0.1, 1.05e-16), (-0.1, -1e-3, 0.99e-16), (-1e-3, 0, 1.08e-16), (0, 1e-3, 1.37e-16), (1e-3, 0.1, 1.22e-16),
          (0.1, 0.5, 1.02e-16), (0.5, 1, 0.77e-16), (1, 2, None), (2, 4, None), (4, 12, None)]


@pytest.mark.parametrize("lo,hi,bound", RANGES, ids=lambda v: str(v))
def test_no_further_off_than_the_library_form(fit, gelu, lo, hi, bound):
    x = np.random.default_rng(3).uniform(lo, hi, 400)

    def true(v):
        t = Decimal(abs(v))
        tail = t * fit.scaled_tail(t) * (-t * t / 2).exp()
        return Decimal(v) - tail if v > 0 else -tail
    want = [true(float(v)) for v in x]
    rms = lambda y: np.sqrt(np.mean([float((Decimal(float(a)) - b) / b) ** 2 for a, b in zip(y, want)]))  # noqa: E731
    if bound is None:
        bound = rms(0.5 * x * erfc(-x * 0.70710678118654752440))
    # 400 samples give a root mean square to a few percent
    assert rms(gelu(x)) <= 1.05 * bound


def test_far_out_and_no_numbers(gelu):
    x = np.array([0.0, 13.0, 39.9, 40.0, 1e10, 1e300, np.inf])
    np.testing.assert_array_equal(gelu(x), x)
    assert (gelu(-x[3:6]) == 0).all() and -1e-313 < gelu(np.array([-38.0]))[0] < 0
    assert np.isnan(gelu(np.array([-np.inf, np.nan]))).all()
