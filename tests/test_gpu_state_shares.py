"""Prompt phase: the state of the discarded pairs from shares of a unit's tokens (GPU, against the oracle).

Sizes around the shares' edges (64 tokens at least to a share, one launch up to 64 tokens), ranks that fill the chunks of eight
rows or not, both storage types.  Tolerances: tests/harness.py.
"""
import pytest

from paper_2402_09398_amd import workloads as wl
from tests.test_gpu_digits import run, shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("prompt,rank,head_dim", [(9, 8, 128), (64, 3, 64), (64, 16, 128), (65, 8, 64), (127, 8, 128), (128, 9, 64),
                                                  (129, 16, 128), (300, 20, 64), (1000, 5, 128)])
def test_shares(prompt, rank, head_dim, dtype):
    w = shape(prompt, rank=rank, head_dim=head_dim, dtype=dtype)
    run(w, wl.all_inputs(w))


@pytest.mark.parametrize("prompt", [70, 71])
def test_inside_and_just_past_the_budget(prompt):
    """Nothing discarded (H = z = 0), one pair discarded."""
    w = shape(prompt, n_heavy=35, n_recent=35)
    run(w, wl.all_inputs(w))
