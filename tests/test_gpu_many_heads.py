"""Decode step with more than eight query heads per key/value head, fp16 storage: the heads as columns
of matrix tiles (GPU, against the oracle).  Head counts around the groups of sixteen, cache sizes at the
edges of the row tiles (16 rows, 8 waves, up to 1024 rows) and beyond them, a cache still filling, the other
options, one block per unit and several.  Tolerances: tests/harness.py."""
import numpy as np
import pytest
import torch

from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


def shape(name, **kw):
    d = dict(name=name, batch=2, heads=1, head_dim=64, prompt=60, steps=8, n_heavy=10, n_recent=10, rank=4, hidden=64,
             dtype="f16", q_per_kv=17)
    d.update(kw)
    return wl.WORKLOADS[2].scaled(**d)


CASES = [
    (shape("heads-9", q_per_kv=9), 0),
    (shape("heads-16-d128", q_per_kv=16, head_dim=128), 0),
    (shape("heads-33-rank-20", q_per_kv=33, rank=20, hidden=48), 0),
    (shape("heads-128", q_per_kv=128, steps=3), 0),
    (shape("one-slot", n_heavy=0, n_recent=1), 0),
    (shape("rows-16", n_heavy=8, n_recent=7), 0),
    (shape("rows-17", n_heavy=8, n_recent=8), 0),
    (shape("rows-128-d128", n_heavy=60, n_recent=67, head_dim=128, prompt=140), 0),
    (shape("rows-129", n_heavy=64, n_recent=64, prompt=140), 0),
    (shape("rows-257-d128", n_heavy=128, n_recent=128, head_dim=128, prompt=300), 0),
    (shape("rows-513", n_heavy=256, n_recent=256, prompt=540, batch=1, steps=4), 0),
    (shape("rows-1024-d128", n_heavy=500, n_recent=523, head_dim=128, prompt=1030, batch=1, steps=4), 0),
    (shape("rows-1024-rank-64-d128", n_heavy=500, n_recent=523, head_dim=128, prompt=1030, batch=1, steps=2, rank=64, hidden=48), 0),
    (shape("rows-1025", n_heavy=512, n_recent=512, prompt=1030, batch=1, steps=4), 0),
    (shape("filling", prompt=0, steps=30), 0),
    (shape("sparse-denominator"), 1),
    (shape("lambda", n_heavy=4), 2),
    (shape("one-block-per-unit", batch=130, heads=4, q_per_kv=18, prompt=30, steps=4), 0),
]


@pytest.mark.parametrize("w,flags", CASES, ids=lambda x: getattr(x, "name", None))
def test_many_heads(w, flags):
    rep = hz.run_workload(w, range(min(w.units, 24)), flags=flags)
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]


def test_values_without_digits():
    """Cached keys and queries with elements of 127 and more: those tiles are multiplied in fp64."""
    w = shape("no-digits", prompt=50, steps=6)
    inp = wl.all_inputs(w)
    inp["K"][:, 45::2, 3] = 300.0
    inp["k"][::2, :, 3] = -150.0
    inp["Q"][..., 3] *= np.float16(1 / 64)
    inp["q"][..., 3] *= np.float16(1 / 64)
    inp["q"][1::3, :, 5, 7] = 200.0
    units = list(range(w.units))
    res = hz.gpu_run(w, inp)
    rep = hz.check_against_oracle(w, inp, units, res)
    rep.failures.extend(hz.check_every_unit(w, res))
    assert rep.ok(), rep.failures[:10]


def test_values_that_cancel():
    """Two keys of nearly the same score with opposite large values: what is left is the difference of their weights,
    1e-6 of each, so weights or sums of 24 bits would leave an error of some percent."""
    w = shape("cancel", prompt=20, steps=1)                 # a full cache, nothing discarded: regular attention
    inp = wl.all_inputs(w)
    for name in "QKVkv":
        inp[name][...] = 0
    inp["K"][:, 3, 0], inp["K"][:, 7, 0] = 1 + 2.0 ** -10, 1
    inp["V"][:, 3], inp["V"][:, 7] = 60000, -60000
    q0 = 2.0 ** -7 * (1 + np.arange(17) / 32)
    inp["q"][...] = 0
    inp["q"][..., 0] = q0
    assert (inp["q"][0, 0, :, 0] == q0).all()
    got = hz.gpu_run(w, inp)["outs"][0].astype(np.float64)  # [U,G,D]
    low = q0 / 8
    exact = 60000 * np.exp(low) * np.expm1(low * 2.0 ** -10) / (np.exp(low) * (2 + np.expm1(low * 2.0 ** -10)) + 19)
    assert (np.abs(got / exact[None, :, None] - 1) < 2.0 ** -10).all(), np.abs(got / exact[None, :, None] - 1).max()


def test_state_that_is_not_finite():
    """An infinite phi(q) z^T: no number comes out, for that unit alone."""
    w = shape("infinite-state", steps=1)
    inp = wl.all_inputs(w)
    gpu = hz.make_gpu(w)
    Q, K, V = (torch.from_numpy(inp[n]).cuda() for n in "QKV")
    gpu.prefill(Q, K, V)
    gpu.z[1] = float("inf")
    q, k, v = (torch.from_numpy(inp[n][0]).cuda() for n in "qkv")
    out = torch.empty_like(q)
    gpu.step(q, k, v, out)
    out = out.cpu().numpy()
    assert np.isnan(out[1]).all() and np.isfinite(out[0]).all()


def test_rows_past_the_last_have_no_value():
    """An infinite element of the step's own value row, which stands in for the rows past the last of a tile: the
    outputs are infinite there, as its weight is not zero, and finite elsewhere."""
    w = shape("infinite-value", steps=1)
    assert (w.capacity + 1) % 16
    inp = wl.all_inputs(w)
    inp["v"][0, :, 7] = np.inf
    out = hz.gpu_run(w, inp)["outs"][0]
    assert np.isposinf(out[..., 7]).all() and np.isfinite(np.delete(out, 7, axis=-1)).all()
