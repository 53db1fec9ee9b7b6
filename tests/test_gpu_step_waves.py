"""Any-shape decode step (fp32 storage, and fp16 shapes that the streaming kernels do not take): row iterations in registers, in the
loop, four or eight waves to a unit (GPU, against the oracle).

Capacities at the edges of the kernel's buckets (2, 4, 7, 11 iterations of four waves; 7, 11, 21 and the loop of eight waves, which few
units take from 12 iterations on; 15, 21 and the loop of four waves with many units), a cache that is still filling, rows of 8, 16 and
32 lanes.  Tolerances: tests/harness.py.
"""
import pytest

from paper_2402_09398_amd import workloads as wl
from tests import harness as hz
from tests.test_gpu_digits import run, shape

pytestmark = pytest.mark.gpu


def run_sample(w, every):
    """All units on the GPU, every so many against the oracle."""
    inp = wl.all_inputs(w, workers=16)
    res = hz.gpu_run(w, inp)
    units = list(range(0, w.units, every)) + [w.units - 1]
    rep = hz.check_against_oracle(w, {k: (v[units] if k in ("Q", "K", "V") else v[:, units]) for k, v in inp.items()}, units, res)
    rep.failures.extend(hz.check_every_unit(w, res))
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]


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


@pytest.mark.parametrize("dtype,head_dim,rank", [("f32", 128, 64), ("f32", 64, 5), ("f16", 128, 20), ("f16", 64, 64)])
@pytest.mark.parametrize("slots", [4000, 4040, 4094])
def test_largest_caches(slots, dtype, head_dim, rank):
    """Up to LESSDEC_MAX_CAPACITY a block's LDS stays within what a launch may take."""
    w = shape(40, steps=2, n_heavy=slots // 2, n_recent=slots - slots // 2, dtype=dtype, head_dim=head_dim, rank=rank)
    run(w, wl.all_inputs(w))


FORMS = {15: 12, 21: 20, 0: 22}                          # four waves: a number of row iterations that takes the form


@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("dtype,head_dim,rank", [("f32", 128, 8), ("f32", 64, 5), ("f16", 128, 20), ("f16", 64, 17)])
def test_four_waves_with_many_units(form, dtype, head_dim, rank):
    """520 units, more than eight waves are taken for: four waves a unit, with the rows of up to 15 or 21 iterations in registers
    or in the loop.  (An iteration is 256 lanes of 16 bytes.)"""
    per = 256 * 16 // (head_dim * (4 if dtype == "f32" else 2))
    slots = FORMS[form] * per - 2
    w = shape(slots + 1, batch=13, heads=40, steps=2, n_heavy=slots // 2, n_recent=slots - slots // 2, dtype=dtype,
              head_dim=head_dim, rank=rank)
    run_sample(w, 37)


@pytest.mark.parametrize("dtype,head_dim,rank", [("f32", 128, 8), ("f16", 64, 17)])
def test_loop_of_eight_waves(dtype, head_dim, rank):
    """260 units, too many for a unit's rows in the registers of eight waves: 12 turns in the loop."""
    slots = 23 * 256 * 16 // (head_dim * (4 if dtype == "f32" else 2)) - 2
    w = shape(slots + 1, batch=13, heads=20, steps=2, n_heavy=slots // 2, n_recent=slots - slots // 2, dtype=dtype,
              head_dim=head_dim, rank=rank)
    run_sample(w, 20)


def test_loop_with_many_units():
    """1040 units keep four waves and the loop."""
    w = shape(190, batch=26, heads=40, steps=2, n_heavy=90, n_recent=90, dtype="f32", rank=8)
    run(w, wl.all_inputs(w, units=None))
