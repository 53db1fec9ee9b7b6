"""Which prompt tokens are kept (GPU, against the oracle): the radix selection of the cheap column sums at its
edges: no heavy slots, all but one token heavy, equal sums, sums that differ in the last bits, prompts around the block
of 256.  Tolerances: tests/harness.py."""
import numpy as np
import pytest

from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


def shape(prompt, heavy, recent, **kw):
    d = dict(name=f"select-{prompt}-{heavy}-{recent}", batch=2, heads=2, head_dim=64, prompt=prompt, steps=2, n_heavy=heavy,
             n_recent=recent, rank=4, hidden=64, dtype="f16")
    d.update(kw)
    return wl.WORKLOADS[2].scaled(**d)


@pytest.mark.parametrize("prompt,heavy,recent,kw", [
    (40, 0, 5, {}), (40, 5, 0, {}), (40, 39, 0, {}), (40, 1, 38, {}), (255, 100, 30, {}), (256, 1, 1, {}), (257, 128, 128, {}),
    (513, 300, 7, dict(head_dim=128)), (700, 50, 50, dict(q_per_kv=3)), (1025, 512, 512, dict(batch=1, heads=1)),
], ids=lambda x: str(x))
def test_kept_set(prompt, heavy, recent, kw):
    w = shape(prompt, heavy, recent, **kw)
    rep = hz.run_workload(w, range(w.units))
    assert rep.ok(), rep.failures[:10]


@pytest.mark.parametrize("spread", [0.0, 1e-3, 0.02])
def test_nearly_equal_sums(spread):
    """Queries of almost zero: every row is nearly uniform, so a token's sum is nearly a function of its position,
    the first ones far apart, the last ones close; with spread 0 exactly so."""
    w = shape(600, 150, 20)
    inp = wl.all_inputs(w)
    inp["Q"][...] = (inp["Q"].astype(np.float32) * spread).astype(np.float16)
    res = hz.gpu_run(w, inp)
    rep = hz.check_against_oracle(w, inp, list(range(w.units)), res)
    rep.failures.extend(hz.check_every_unit(w, res))
    assert rep.ok(), rep.failures[:10]


@pytest.mark.parametrize("prompt,heavy,recent,kw", [
    (64, 32, 32, {}), (64, 6, 6, {}), (40, 14, 14, {}), (130, 65, 65, dict(head_dim=128)), (257, 30, 30, {}),
    (120, 10, 20, dict(q_per_kv=4, head_dim=128)), (460, 20, 20, {}), (460, 240, 240, dict(head_dim=128)),
    (450, 60, 60, dict(heads=24)), (500, 40, 30, dict(heads=24, batch=33)),
], ids=lambda x: str(x))
def test_kept_set_of_many_units(prompt, heavy, recent, kw):
    """256 units and more: the forms of the exact column sums for short and for long sweeps, by the number of key tiles."""
    w = shape(prompt, heavy, recent, **{**dict(batch=32, heads=8), **kw})
    rep = hz.run_workload(w, [0, 1, 100, w.units // 2 + 5, w.units - 1])
    assert rep.ok(), rep.failures[:10]
