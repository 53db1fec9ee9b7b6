"""What a step of many query heads (or of fp32 storage with several) does once the heads are through: the choice of the pair that leaves over
several waves' rows, its fold into H in one pass and in several, the new pair's row, in the step's own block and in a launch of its own;
against the oracle (GPU; tolerances: tests/harness.py)."""
import pytest

from paper_2402_09398_amd import binding
from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


def shape(name, units, g, slots, **kw):
    d = dict(name=name, batch=units, heads=1, head_dim=64, prompt=slots, steps=6, n_heavy=slots // 2, n_recent=slots - slots // 2, rank=8,
             hidden=64, dtype="f16", q_per_kv=g)
    d.update(kw)
    return wl.WORKLOADS[2].scaled(**d)


@pytest.mark.parametrize("w,flags", [
    (shape("oldest-of-several-waves", 2, 17, 140, n_heavy=4, n_recent=136, steps=150), binding.FLAG_LAMBDA),   # equal scores: every slot's turn
    (shape("new-pair-leaves", 2, 17, 70, n_heavy=70, n_recent=0), 0),
    (shape("one-element-rank", 2, 9, 5, rank=1), 0),
    (shape("fold-of-two-passes", 2, 16, 30, head_dim=128, rank=33, hidden=48), 0),
    (shape("own-block-512-threads", 260, 16, 20, steps=4), 0),
    (shape("own-block-two-passes", 260, 16, 20, steps=3, head_dim=128, rank=40, hidden=48), 0),
    (shape("f32-own-block", 300, 3, 70, dtype="f32", steps=4), 0),
    (shape("f32-own-launch", 2, 12, 70, dtype="f32", head_dim=128), 0),
    (shape("f32-unstaged", 2, 5, 600, dtype="f32", head_dim=128, prompt=610, steps=3, rank=20, hidden=48), 0),
    (shape("f32-filling", 3, 4, 40, dtype="f32", prompt=0, steps=50), 0),
    (shape("f32-new-pair-leaves", 3, 4, 40, dtype="f32", n_heavy=40, n_recent=0), 0),
], ids=lambda x: x.name if hasattr(x, "name") else f"flags{x}")
def test_against_oracle(w, flags):
    rep = hz.run_workload(w, sorted({0, 1, w.units // 2, w.units - 1}), flags=flags)
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]
