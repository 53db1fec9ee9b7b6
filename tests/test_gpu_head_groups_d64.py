"""Decode step, fp16, two to eight query heads per unit of 64 elements: the forms for ranks up to 8 and for more, by rows a lane, heads a wave and
where the maps come from, against the oracle (GPU; tolerances: tests/harness.py)."""
import pytest

from tests import harness as hz
from tests.test_gpu_head_groups import shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g", [2, 3, 8])
@pytest.mark.parametrize("slots,rank,hidden", [(90, 8, 64), (127, 9, 64), (128, 7, 64), (255, 16, 64), (256, 8, 64), (300, 12, 640), (20, 1, 640)])
def test_against_oracle(g, slots, rank, hidden):
    w = shape((2, 3), g, slots, rank=rank, hidden=hidden, head_dim=64, steps=5)
    rep = hz.run_workload(w, range(0, w.units, 2))
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]


def test_many_units():
    """Three heads and more units than small launches have: waves of two heads."""
    w = shape((65, 4), 3, 150, head_dim=64, steps=4)
    rep = hz.run_workload(w, [0, 5, w.units - 1])
    assert rep.ok(), rep.failures[:10]


@pytest.mark.parametrize("g", [2, 3, 5, 6])
@pytest.mark.parametrize("slots,rank", [(3, 9), (33, 16), (63, 12), (64, 16), (65, 10), (126, 16)])
def test_ring_of_four(g, slots, rank):
    """Ranks above 8 and up to 128 rows: two heads a wave in most of these; 32 rows of a unit make a pass of a wave of two."""
    w = shape((65, 4) if g > 2 else (2, 3), g, slots, rank=rank, head_dim=64, steps=5)
    rep = hz.run_workload(w, sorted({0, 1, w.units // 2, w.units - 1}))
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]
