"""Prompt phase with fp16 storage: scores from digit planes of the halves (GPU, against the oracle).

Sizes at the edges of the tiles (16 queries per wave, 32 keys per tile, 64 or 128 queries per
workgroup), values that have no digits (|x| >= 127: those tiles are multiplied in fp64) and values that
are not finite.  Tolerances: tests/harness.py.
"""
import numpy as np
import pytest

from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


def shape(prompt, **kw):
    d = dict(name=f"digits-{prompt}", batch=1, heads=3, head_dim=128, prompt=prompt, steps=2, n_heavy=4, n_recent=4,
             rank=4, hidden=64, dtype="f16")
    d.update(kw)
    return wl.WORKLOADS[2].scaled(**d)


def run(w, inp):
    units = list(range(w.units))
    res = hz.gpu_run(w, inp)
    rep = hz.check_against_oracle(w, inp, units, res)
    rep.failures.extend(hz.check_every_unit(w, res))
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]
    return res


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("prompt", [1, 9, 16, 17, 31, 32, 33, 48, 63, 64, 65, 97, 128, 129, 161])
def test_tile_edges(prompt, head_dim):
    w = shape(prompt, head_dim=head_dim)
    run(w, wl.all_inputs(w))


def test_long_prompt():
    """A prompt of many key tiles that ends inside one."""
    w = shape(4096 + 37, heads=1)
    run(w, wl.all_inputs(w))


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("which", ["K", "Q", "KQ"])
def test_values_without_digits(which, head_dim):
    """Some rows carry elements of 127 and more (and the largest that still has digits, 126.9)."""
    w = shape(150, head_dim=head_dim, q_per_kv=2)
    inp = wl.all_inputs(w)
    rng = np.random.default_rng(5)
    for name in which:
        x = inp[name].reshape(w.units, -1, w.prompt, head_dim)
        for value in (126.9375, -126.9375, 127.0, -300.0, 6e4 if which == "K" else 900.0):
            for u in range(w.units):
                for head in range(x.shape[1]):
                    x[u, head, rng.integers(2, w.prompt), rng.integers(head_dim)] = value
    # what the large channel meets is small, so that the rows stay soft
    other = {"K": "Q", "Q": "K"}.get(which)
    if other:
        big = np.abs(inp[which].astype(np.float32)).reshape(-1, head_dim).max(axis=0) > 100
        inp[other][..., big] *= np.float16(1 / 64)
    run(w, inp)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_rows_before_a_value_that_is_not_finite(value):
    """Rows of earlier tiles neither see the key nor its value: bit for bit as without it."""
    w = shape(100, steps=0)
    clean = wl.all_inputs(w)
    dirty = {k: v.copy() for k, v in clean.items()}
    dirty["K"][:, 70, 5] = value
    dirty["V"][:, 70, 7] = value
    a, b = (hz.gpu_run(w, x)["prefill_out"] for x in (clean, dirty))
    assert np.array_equal(a[:, :64].view(np.uint16), b[:, :64].view(np.uint16))


@pytest.mark.parametrize("before,after", [(20, 40), (36, 50), (20, 50), (3, 20)])
@pytest.mark.parametrize("low,high", [(10.0, 17.5), (10.0, 25.0), (9.0, 11.0)])
def test_maximum_that_jumps(before, after, low, high):
    """A weight just below the limit for moving the maximum, not yet multiplied with its value when a far larger
    score moves it: it keeps its share (e^(low - high), with a value that makes it visible)."""
    w = shape(70, head_dim=64)
    inp = wl.all_inputs(w)
    inp["Q"][...] = 0
    inp["Q"][..., 0] = 8.0                               # score = first element of the key
    inp["K"][..., 0] = 0.0
    inp["K"][:, before, 0] = low
    inp["K"][:, after, 0] = high
    inp["V"][:, before, :] = 300.0
    run(w, inp)


@pytest.mark.parametrize("prompt", [65, 79, 81, 95])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_last_tile_reads_nothing_of_the_next_unit(prompt, value):
    """A prompt that ends inside a tile of 32 keys: rows past it, which are the next unit's first, have no part in
    the last queries' outputs, whatever they hold (a weight of zero would still make NaN of them)."""
    w = shape(prompt, steps=0)
    clean = wl.all_inputs(w)
    dirty = {k: v.copy() for k, v in clean.items()}
    for name in "KV":
        dirty[name][1:, :20] = value
    a, b = (hz.gpu_run(w, x)["prefill_out"] for x in (clean, dirty))
    assert np.array_equal(a[0].view(np.uint16), b[0].view(np.uint16))


@pytest.mark.parametrize("which", ["K", "Q"])
def test_values_without_digits_keep_the_speed_of_fp64_products(which):
    """One channel of 200 in every row sends every tile to the fp64 matrix unit.  A 16 x 16 tile is D / 4 products of 66
    cycles there against D / 4 of 16 with digits, and the rest of a tile (weights, values, staging) is the same: at
    most 66 / 16 times the clean prompt's time even if nothing else counted, two times measured.  Bound: 3."""
    import torch
    w = shape(1024, batch=16, heads=16, steps=0, n_heavy=51, n_recent=51, rank=8, hidden=512)
    gpu = hz.make_gpu(w)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = {n: torch.randn(w.units, w.prompt, w.head_dim, generator=g, device="cuda").half() for n in "QKV"}
    out = torch.empty_like(x["Q"])

    def ms():
        times = []
        for _ in range(7):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            gpu.prefill(x["Q"], x["K"], x["V"], out=out)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[2]

    clean = ms()
    x[which][..., 3] = 200.0
    x["KQ".replace(which, "")][..., 3] *= 1 / 64
    large = ms()
    print(f"\nclean {clean:.3f} ms, with a channel of 200 in {which} {large:.3f} ms", flush=True)
    assert large < 3 * clean


def test_small_weights_keep_their_bits():
    """Weights near the floor of the fp16 pairs that p V takes: relative to the row's largest weight none is off by more
    than 2^-25 (half a step of the halves below 2^-14, for a largest weight of 1).  Keys of two scores: one of the
    largest, a little above an integer in base-2 units, with value 0, and many 24 octaves below it with value 60000."""
    w = shape(64, head_dim=64, heads=1, steps=0)
    top = np.arange(8, 16, 2.0 ** -7)
    top = top[(top / np.log(2) % 1 > 0.002) & (top / np.log(2) % 1 < 0.02)]
    low = np.arange(-8, -4, 2.0 ** -8)
    gap = (top[:, None] - low[None, :]) / np.log(2) - 24 - top[:, None] / np.log(2) % 1
    i, j = np.argwhere((gap > 0.002) & (gap < 0.02))[0]
    inp = wl.all_inputs(w)
    inp["Q"][...] = 0
    inp["Q"][..., 0] = 8.0                               # score = first element of the key
    inp["K"][...] = 0
    inp["K"][..., 0] = low[j]
    inp["K"][:, 0, 0] = top[i]
    inp["V"][...] = 60000.0
    inp["V"][:, 0] = 0
    assert inp["K"][0, 0, 0] == top[i] and inp["K"][0, 1, 0] == low[j]
    got = hz.gpu_run(w, inp)["prefill_out"].astype(np.float64)[0]
    n = np.arange(w.prompt)[:, None]                     # query n sees n of the small ones
    r = np.exp(low[j] - top[i])
    exact = n * r * 60000 / (1 + n * r)
    assert (np.abs(got - exact) <= n * 2.0 ** -25 * 60000 + exact * 2.0 ** -10).all(), np.abs(got - exact).max() / exact.max()


@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_row_without_a_log_sum_has_no_part_in_column_sums(value):
    """An infinite query element: its row's scores are infinite and the row has no log-sum.  The column sums are
    those of the other rows (its own weights are not numbers), and whatever they decide stays decidable."""
    w = shape(100, steps=0)
    inp = wl.all_inputs(w)
    inp["Q"][0, 40, 5] = value
    acc, pos = (hz.gpu_run(w, inp)["after_prefill"][n][0] for n in ("acc", "pos"))
    s = inp["Q"][0].astype(np.float64) @ inp["K"][0].astype(np.float64).T / np.sqrt(w.head_dim)
    s[40] = 0
    a = np.exp(np.where(np.tril(np.ones_like(s, dtype=bool)), s, -np.inf))
    a /= a.sum(1, keepdims=True)
    a[40] = 0
    assert np.isfinite(acc).all() and np.allclose(acc, a.sum(0)[pos], rtol=1e-6, atol=0)
