"""Decode step, fp16, maps with more than eight parts (hidden widths above 512): the parts past the eighth in rounds of four, whole and ragged,
for a unit over one, two, four and eight waves, every form (rows a lane, rank, head_dim), against the oracle (GPU; tolerances:
tests/harness.py)."""
import pytest

from tests import harness as hz
from tests.test_gpu_split_roles import shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [544, 768, 800, 1056, 2048])       # 9, 12, 13, 17 and 32 parts
@pytest.mark.parametrize("units,slots,head_dim,rank", [
    ((2, 3), 20, 128, 8), ((2, 3), 50, 64, 5),                         # a wave: few rows
    ((2, 3), 40, 128, 16), ((2, 3), 100, 128, 8), ((2, 3), 200, 64, 9), ((2, 3), 200, 128, 3), ((2, 3), 300, 128, 12),
])
def test_against_oracle(units, slots, head_dim, rank, hidden):
    w = shape(units, slots, head_dim=head_dim, rank=rank, hidden=hidden, steps=4)
    rep = hz.run_workload(w, [0, w.units - 1])
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]


@pytest.mark.parametrize("units,slots", [((200, 8), 130), ((100, 10), 70)])     # a wave per unit, two
def test_many_units(units, slots):
    w = shape(units, slots, hidden=1056, steps=3)
    rep = hz.run_workload(w, [0, w.units // 2, w.units - 1])
    assert rep.ok(), rep.failures[:10]
