"""Derives the constants of gelu_poly_f64() in lessdec_common.h.

Upper tail of the standard normal, Q(t) = 0.5 erfc(t / sqrt 2), t >= 0, is written as
Q(t) = exp(-t^2 / 2) * sum_{k=1..7} c_k u^k with u = 1 / (1 + p t): exp(t^2/2) Q(t) is a smooth,
slowly decaying function of t and a low-degree polynomial in u captures it to 1e-9.  Then
gelu(x) = x - |x| Q(|x|) for x >= 0 and -|x| Q(|x|) for x < 0.  Weighted least squares on a
dense grid (the weight is the factor exp(-t^2/2) t that multiplies the polynomial's error in
gelu).  Prints p, c_1..c_7 and the error of a float32 evaluation against float64 erfc, the measure
of the form below.

And those of gelu_exp2_f32(): log2 Q(t) = c_0 + c_1 s + ... + c_10 s^10, s = t - 1, so that gelu takes one base-2
exponential and no reciprocal: near-minimax (Lawson's reweighted least squares) in the relative error of Q, which may
grow tenfold per unit beyond t = 3, as that of the form above does, and counts for less where t Q(t) falls below 1e-9.  The
coefficients are rounded to fp32 one after the other, lowest first, and the others fitted again.
"""
import numpy as np
from scipy.special import erfc, erfcx, log_ndtr

P, N = 0.24, 7
CENTRE, DEGREE = 1.0, 10


def fit(p=P, n=N):
    t = np.concatenate([np.linspace(0, 8, 20001), np.linspace(8, 14, 2001)])
    u = 1 / (1 + p * t)
    target = 0.5 * erfcx(t / np.sqrt(2))                    # exp(t^2/2) Q(t), computed stably
    A = np.stack([u ** k for k in range(1, n + 1)], axis=1)
    w = np.exp(-t * t / 2) * np.maximum(t, 0.5)
    c, *_ = np.linalg.lstsq(A * w[:, None], target * w, rcond=None)
    return c


def _fma(a, b, c):
    """Fused multiply-add of fp32 values, rounded to fp32 (the product is exact in fp64, the sum all but)."""
    return (a.astype(np.float64) * b + c).astype(np.float32)


def gelu32(x, p, c):
    """With the reciprocal, in fp32: what gelu_exp2_f32 is measured by."""
    x = x.astype(np.float32)
    c = [np.float32(v) for v in c]
    t = np.abs(x)
    u = np.float32(1) / _fma(t, np.float32(p), 1.0)
    acc = np.full_like(u, c[-1])
    for k in range(len(c) - 2, -1, -1):
        acc = _fma(acc, u, c[k])
    e = np.exp2((t * t * np.float32(-0.5 * np.log2(np.e))).astype(np.float64)).astype(np.float32)
    return np.maximum(x, 0) - t * (acc * u * e)


def fit_log2(n=DEGREE, centre=CENTRE, top=7.5, rounds=300):
    """c_0 .. c_n, each of them a fp32 number, and the largest weighted error before the rounding."""
    t = (top * (0.5 - 0.5 * np.cos(np.linspace(0, np.pi, 4001))))[1:]
    y, tq = log_ndtr(-t) / np.log(2), t * np.exp(log_ndtr(-t))
    w = np.log(2) * tq / np.maximum(tq * 1e-7 * 10 ** np.maximum(t - 3, 0), 2e-13)
    A = ((t - centre)[:, None] / top) ** np.arange(n + 1)

    def solve(lam, known):
        r = np.sqrt(lam) * w
        k = len(known)
        rest = y - A[:, :k] @ (np.array(known) * top ** np.arange(k))
        c, *_ = np.linalg.lstsq(A[:, k:] * r[:, None], rest * r, rcond=None)
        return c / top ** np.arange(k, n + 1), np.abs((A[:, k:] @ c - rest) * w)

    lam, best = np.full_like(t, 1 / len(t)), None
    for _ in range(rounds):
        c, e = solve(lam, [])
        if best is None or e.max() < best[0]:
            best = (e.max(), lam)
        lam = lam * e / (lam * e).sum()
    known = []
    while len(known) <= n:
        known.append(float(np.float32(solve(best[1], known)[0][0])))
    return known, best[0]


def gelu_exp2_32(x, c, centre=CENTRE):
    """As the kernels evaluate it."""
    x = x.astype(np.float32)
    t = np.abs(x)
    s = t - np.float32(centre)
    p = np.full_like(t, np.float32(c[-1]))
    for k in range(len(c) - 2, -1, -1):
        p = _fma(p, s, np.float32(c[k]))
    e = np.exp2(p.astype(np.float64)).astype(np.float32)
    return (np.maximum(x, 0).astype(np.float64) - t.astype(np.float64) * e).astype(np.float32)


if __name__ == "__main__":
    c = fit()
    print("p =", P)
    for k, v in enumerate(c, 1):
        print(f"c{k} = {v:.10e}")
    x = np.linspace(-12, 12, 2000001)
    exact = 0.5 * x * erfc(-x / np.sqrt(2))
    err = np.abs(gelu32(x, P, c).astype(np.float64) - exact)
    print("max abs error on [-12, 12]:", err.max(), "; on [-4, 4]:", err[np.abs(x) <= 4].max())
    print("max error / max(|gelu|, |x| 6e-8, 1e-30):", (err / np.maximum(np.abs(exact), 1e-30))[np.abs(x) > 1e-3].max())
    c10, worst = fit_log2()
    print("log2 Q about", CENTRE, ":", ", ".join(f"{v:.10e}" for v in c10), "; of the allowed error", worst)
    e10 = np.abs(gelu_exp2_32(x, c10).astype(np.float64) - exact)
    for lo, hi in ((-6, -5), (-5, -4), (-4, -3), (-3, -2), (-2, -1), (-1, 0), (0, 1), (1, 2), (2, 4)):
        k = (x >= lo) & (x <= hi)
        print([lo, hi], "root mean square with the reciprocal", np.sqrt((err[k] ** 2).mean()), "; exp2", np.sqrt((e10[k] ** 2).mean()))
