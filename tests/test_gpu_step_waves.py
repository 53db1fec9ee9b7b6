"""Any-shape decode step (fp32 storage, and fp16 shapes that the streaming kernels do not take): row iterations in registers, in the
loop, four or eight waves to a unit (GPU, against the oracle).

Capacities at the edges of the kernel's buckets (2, 4, 7, 11, 15, 21 iterations of 8 or 16 rows; eight waves from 12 on), a cache that
is still filling, rows of 8, 16 and 32 lanes.  Tolerances: tests/harness.py.
"""
import pytest

from paper_2402_09398_amd import workloads as wl
from tests.test_gpu_digits import run, shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,head_dim,rank", [("f32", 128, 8), ("f32", 64, 5), ("f16", 128, 20), ("f16", 64, 17)])
@pytest.mark.parametrize("slots", [15, 16, 31, 32, 56, 87, 88, 119, 175, 176, 335, 336, 351, 700])
def test_capacities(slots, dtype, head_dim, rank):
    w = shape(slots + 2, steps=3, n_heavy=slots // 2, n_recent=slots - slots // 2, dtype=dtype, head_dim=head_dim, rank=rank)
    run(w, wl.all_inputs(w))


@pytest.mark.parametrize("slots", [100, 400])
def test_filling(slots):
    """Prompt shorter than the cache: the appended pair's row lies inside the requested ones."""
    w = shape(slots // 2, steps=4, n_heavy=slots // 2, n_recent=slots // 2, dtype="f32", rank=8)
    run(w, wl.all_inputs(w))


def test_four_waves_with_many_units():
    """1040 units keep four waves and the loop."""
    w = shape(190, batch=26, heads=40, steps=2, n_heavy=90, n_recent=90, dtype="f32", rank=8)
    run(w, wl.all_inputs(w, units=None))
