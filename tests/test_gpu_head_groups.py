"""Decode step, fp16, two to eight query heads per unit: waves of two and of four heads, which share a unit's rows, on both sides of the rule
between them; odd head counts, ragged and tiny caches, every form (rows a lane, rank, head_dim, one launch or two), a filling cache, an
empty window, both policies and denominators, against the oracle (GPU; tolerances: tests/harness.py)."""
import pytest

from paper_2402_09398_amd import binding
from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


def shape(units, g, slots, **kw):
    batch, heads = units
    d = dict(name=f"heads-{batch}x{heads}x{g}-{slots}", batch=batch, heads=heads, head_dim=128, prompt=slots + 5, steps=8, n_heavy=slots // 2,
             n_recent=slots - slots // 2, rank=8, hidden=64, dtype="f16", q_per_kv=g)
    d.update(kw)
    return wl.WORKLOADS[2].scaled(**d)


@pytest.mark.parametrize("w,flags", [
    (shape((3, 2), 2, 1, n_heavy=0, n_recent=1), 0), (shape((3, 2), 2, 3), 0), (shape((3, 2), 4, 4, rank=5), 0),
    (shape((2, 3), 2, 127), 0), (shape((2, 3), 2, 128, rank=12), 0), (shape((2, 2), 3, 255), 0), (shape((2, 2), 4, 256, steps=5), 0),
    (shape((2, 2), 5, 70, rank=16), binding.FLAG_SPARSE_DENOM), (shape((2, 2), 6, 300, steps=5), 0), (shape((2, 2), 7, 33), 0),
    (shape((2, 2), 8, 511, steps=4), 0), (shape((1, 2), 8, 129, rank=11), 0),
    (shape((2, 2), 4, 60, head_dim=64), 0), (shape((2, 2), 3, 200, head_dim=64, rank=3), 0), (shape((2, 1), 7, 260, head_dim=64, steps=5), 0),
    (shape((2, 2), 8, 40, prompt=30, steps=25), 0),                   # filling, then full, one launch
    (shape((2, 2), 4, 50, n_heavy=50, n_recent=0), 0),                # the new pair may be the one that leaves
    (shape((2, 2), 6, 50, n_heavy=50, n_recent=0), binding.FLAG_LAMBDA),
    (shape((2, 2), 4, 150, n_heavy=4, n_recent=146), binding.FLAG_LAMBDA),
    (shape((64, 4), 3, 20, steps=5), 0), (shape((65, 4), 3, 20, steps=5), 0),       # 1024 waves, and more
    (shape((32, 4), 5, 20, steps=5), 0), (shape((33, 4), 5, 20, steps=5), 0),
], ids=lambda x: f"{x.name}-{x.head_dim}-{x.rank}-{x.n_recent}" if hasattr(x, "name") else f"flags{x}")
def test_against_oracle(w, flags):
    rep = hz.run_workload(w, sorted({0, 1, w.heads, w.units // 2, w.units - 1} & set(range(w.units))), flags=flags)
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]
