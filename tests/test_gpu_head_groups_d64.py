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
