"""The state a prompt leaves (GPU, against the oracle): slots, gathered rows, H and z of the discarded pairs, at ranks
around the chunk of eight rows, ragged prompts, both storage types; and the prefix states of Lambda-masking through the
prompt at prompts around the block of 64 keys.  Tolerances: tests/harness.py."""
import numpy as np
import pytest

from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


def shape(**kw):
    d = dict(name="prompt-state", batch=1, heads=3, head_dim=128, prompt=131, steps=3, n_heavy=5, n_recent=6, rank=8, hidden=64,
             dtype="f16")
    d.update(kw)
    return wl.WORKLOADS[2].scaled(**d)


@pytest.mark.parametrize("kw", [
    dict(rank=1, hidden=32), dict(rank=7), dict(rank=8), dict(rank=9), dict(rank=16), dict(rank=64, hidden=48),
    dict(prompt=12), dict(prompt=33, head_dim=64), dict(prompt=700, head_dim=64, rank=12), dict(dtype="f32", rank=5),
    dict(dtype="f32", head_dim=64, rank=10, prompt=70), dict(prompt=8, n_heavy=8, n_recent=8), dict(prompt=1500, n_heavy=600, n_recent=300),
    dict(prompt=256), dict(prompt=257), dict(prompt=300, dtype="f32", rank=9),
], ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
def test_state(kw):
    w = shape(**kw)
    rep = hz.run_workload(w, range(w.units))
    assert rep.ok(), rep.failures[:10]


@pytest.mark.parametrize("kw", [
    dict(prompt=40, n_heavy=4, n_recent=8), dict(prompt=63, n_heavy=4, n_recent=8), dict(prompt=64, n_heavy=4, n_recent=8),
    dict(prompt=129, n_heavy=4, n_recent=20), dict(prompt=300, n_heavy=70, n_recent=9, rank=16),
    dict(prompt=260, n_heavy=4, n_recent=30, rank=13, head_dim=64), dict(prompt=200, n_heavy=4, n_recent=10, dtype="f32", rank=3),
], ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
def test_prefix_states(kw):
    w = shape(**kw)
    rep = hz.run_workload(w, range(w.units), flags=2 | 4)
    assert rep.ok(), rep.failures[:10]


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_kept_tokens_that_are_not_finite(dtype):
    """Kept tokens have no part in H and z, whatever their psi and values are (Lambda-masking: the kept set does not
    depend on them)."""
    w = shape(dtype=dtype, steps=0)
    clean = wl.all_inputs(w)
    dirty = {k: v.copy() for k, v in clean.items()}
    dirty["K"][:, -1, 5] = np.nan
    dirty["V"][:, -2, 7] = np.inf
    a, b = (hz.gpu_run(w, x, flags=2)["after_prefill"] for x in (clean, dirty))
    assert np.isnan(b["psi"]).any()
    for name in ("H", "z"):
        assert np.array_equal(a[name], b[name]), name
