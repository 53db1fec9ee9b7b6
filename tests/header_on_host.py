"""Functions of csrc/lessdec_common.h run on the CPU: their text as it stands in the header, compiled for the host with the few
instructions that C++ does not have replaced (1 / d to 24 bits for the fp64 reciprocal, 2^x rounded once for the fp32 one)."""
import ctypes
import re
import subprocess
import tempfile
from pathlib import Path

import numpy as np

CSRC = Path(__file__).resolve().parents[1] / "paper_2402_09398_amd" / "csrc"
SHIMS = """#include <cmath>
#define __device__
static inline double __builtin_amdgcn_rcp(double d) { return (double)(float)(1.0 / d); }
static inline float __builtin_amdgcn_exp2f(float x) { return (float)std::exp2((double)x); }
using std::fma; using std::fmaf; using std::exp; using std::fabs;
"""


def body(name):
    """The function's text, from its return type to the closing brace."""
    src = (CSRC / "lessdec_common.h").read_text()
    at = src.index(f" {name}(")
    at = src.rindex("__device__", 0, at + 1)
    return src[at:src.index("\n}\n", at) + 3]


def horner(text, name, arg):
    """Coefficients of `name` as a polynomial in `arg`, highest first, as written in the function's text."""
    number = r"(-?[\d.]+(?:e[-+]\d+)?)f?"
    first = float(re.search(rf"{name} = {number};", text).group(1))
    return [first] + [float(x) for x in re.findall(rf"{name} = fmaf?\({name}, {arg}, {number}\);", text)]


def _with_callees(names):
    """These functions and the header's own that they call, callees first."""
    src = (CSRC / "lessdec_common.h").read_text()
    known = re.findall(r"^__device__ inline \w+ (\w+)\(", src, re.M)
    out = []

    def add(name):
        for other in known:
            if other != name and re.search(rf"\b{other}\(", body(name)):
                add(other)
        if name not in out:
            out.append(name)
    for n in names:
        add(n)
    return out


def on_host(*names):
    """name -> function of an array, for functions of one argument."""
    kinds = {n: body(n).split("inline ")[1].split()[0] for n in names}
    with tempfile.TemporaryDirectory() as tmp:
        text = SHIMS + "".join(body(n) for n in _with_callees(names))
        for n, t in kinds.items():
            text += f'extern "C" void run_{n}(const {t} *x, {t} *y, long n) {{ for (long i = 0; i < n; ++i) y[i] = {n}(x[i]); }}\n'
        (Path(tmp) / "f.cpp").write_text(text)
        subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-fPIC", "-shared", "-o", f"{tmp}/f.so", f"{tmp}/f.cpp"],
                       check=True)
        lib = ctypes.CDLL(f"{tmp}/f.so")

    def caller(n):
        dtype = np.float32 if kinds[n] == "float" else np.float64

        def call(x):
            x = np.ascontiguousarray(x, dtype)
            y = np.empty_like(x)
            getattr(lib, f"run_{n}")(x.ctypes.data_as(ctypes.c_void_p), y.ctypes.data_as(ctypes.c_void_p), ctypes.c_long(x.size))
            return y
        return call
    return {n: caller(n) for n in names}
