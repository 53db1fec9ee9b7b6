"""Decode step, fp16, a unit's rows over two, four and eight waves, which share out the work behind the scores: every form (rows a lane,
rank, head_dim, one launch or two) with a full and a filling cache, the window empty (the new pair itself may leave) and both
policies, against the oracle (GPU; tolerances: tests/harness.py)."""
import pytest

from paper_2402_09398_amd import binding
from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


def shape(units, slots, **kw):
    batch, heads = units
    d = dict(name=f"roles-{batch}x{heads}-{slots}", batch=batch, heads=heads, head_dim=128, prompt=slots + 9, steps=10, n_heavy=slots // 2,
             n_recent=slots - slots // 2, rank=8, hidden=64, dtype="f16")
    d.update(kw)
    return wl.WORKLOADS[2].scaled(**d)


@pytest.mark.parametrize("w,flags", [
    (shape((100, 10), 70), 0),                                        # two waves
    (shape((100, 10), 130, rank=16, steps=6), 0),
    (shape((60, 16), 300, head_dim=64, steps=6), 0),
    (shape((3, 5), 63), 0),                                           # four, one row a lane more and less than 64
    (shape((3, 5), 64, rank=3), binding.FLAG_SPARSE_DENOM),
    (shape((3, 5), 64, prompt=50, steps=30), 0),                      # filling, then full
    (shape((3, 5), 90, n_heavy=90, n_recent=0), 0),                   # the new pair may be the one that leaves
    (shape((3, 5), 90, n_heavy=4, n_recent=86), binding.FLAG_LAMBDA),
    (shape((3, 5), 90, n_heavy=90, n_recent=0), binding.FLAG_LAMBDA),
    (shape((2, 7), 127), 0), (shape((2, 7), 128), 0),                 # eight; the forms' edges
    (shape((2, 7), 255, rank=13), 0), (shape((2, 7), 256, prompt=250, steps=20), 0), (shape((2, 7), 511, steps=4), 0),
    (shape((2, 7), 200, head_dim=64, rank=6), binding.FLAG_SPARSE_DENOM),
    (shape((70, 7), 260, steps=6), binding.FLAG_LAMBDA),              # four, more than 256 rows
], ids=lambda x: f"{x.name}-{x.head_dim}-{x.rank}-{x.n_recent}" if hasattr(x, "name") else f"flags{x}")
def test_against_oracle(w, flags):
    rep = hz.run_workload(w, sorted({0, 1, w.heads, w.units // 2, w.units - 1}), flags=flags)
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]
