"""The fp64 exponential of the softmax weights: the constants typed into csrc/lessdec_digits.h are the ones that
csrc/fit_exp2_poly.py derives, and evaluated as the kernels evaluate them they stay within the error the header
states."""
import importlib.util
import re
from pathlib import Path

import numpy as np

CSRC = Path(__file__).resolve().parents[1] / "paper_2402_09398_amd" / "csrc"


def _fit_module():
    spec = importlib.util.spec_from_file_location("fit_exp2_poly", CSRC / "fit_exp2_poly.py")
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def _header_constants():
    """c0 .. c9 as written in exp2_f64 (the leading one apart, the others in Horner order)."""
    src = (CSRC / "lessdec_digits.h").read_text()
    body = src[src.index("inline void exp2_f64"):]
    body = body[:body.index("\n}\n")]
    rest = re.search(r"kPoly\[9\] = \{(.*?)\}", body, re.S).group(1)
    lead = re.search(r"p\[i\] = (\d\.\d+e-\d+);", body).group(1)
    return [float(x) for x in [lead] + rest.split(",")][::-1]


def test_header_constants_are_the_derived_ones():
    fit = _fit_module()
    assert fit.fit() == _header_constants() and len(_header_constants()) == fit.DEGREE + 1


def test_error():
    fit = _fit_module()
    y = np.concatenate([np.linspace(-40, 15, 400001), np.linspace(-1000, -40, 100001)])
    n = np.rint(y)
    got = np.ldexp(fit.evaluate(_header_constants(), y - n), n.astype(int))
    assert np.abs(got / np.exp2(y.astype(np.longdouble)) - 1).max() < 1.9e-14
