"""Prompt phase, fp16: psi of the keys in the row pass's launch or in one of its own, on both sides of the lines for full blocks of maps with
short sweeps, for long sweeps and for head_dim 64 (GPU).  The same bits, see tests/test_gpu_maps_ride.py."""
import pytest

from tests.test_gpu_maps_ride import test_both_sides_of_the_line as both_sides

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,rank,hidden,heads,prompt,batches", [
    (128, 8, 512, 16, 130, (78, 80)),                    # 2560 at R' = 512 and rank 8, ragged rows
    (128, 16, 512, 32, 64, (80, 81)),                    # 2560
    (128, 8, 512, 16, 520, (47, 48)),                    # 6144 with sweeps of more than eight workgroups
    (64, 8, 512, 32, 64, (128, 129)),                    # 4096 at D = 64
])
def test_lines(head_dim, rank, hidden, heads, prompt, batches):
    both_sides(head_dim, rank, hidden, heads, prompt, batches)
