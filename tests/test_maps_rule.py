"""The rule by which psi of a prompt's keys rides in the row pass's launch (CPU)."""
import pytest

from tests import test_gpu_maps_ride, test_gpu_maps_ride_lines
from tests.maps_rule import rides


def _cases(test):
    return next(m for m in test.pytestmark if m.name == "parametrize").args[1]


@pytest.mark.parametrize("head_dim,rank,hidden,heads,prompt,batches",
                         _cases(test_gpu_maps_ride.test_both_sides_of_the_line) + _cases(test_gpu_maps_ride_lines.test_lines))
def test_the_gpu_cases_lie_on_both_sides(head_dim, rank, hidden, heads, prompt, batches):
    """Where the rule moves, the cases that compare its two ways have to move with it."""
    assert [rides(b, heads, prompt, head_dim, hidden, rank) for b in batches] == [True, False]
    assert batches[1] - batches[0] == 1


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("hidden,rank", [(128, 8), (256, 4), (384, 8), (512, 5), (512, 8), (512, 16), (96, 8), (1024, 8)])
def test_monotone(head_dim, hidden, rank):
    """More prompts of one length never bring psi back into the launch, and longer sweeps never take it out at as many workgroups of maps."""
    last = 0
    for sweep in (1, 2, 3, 4, 8, 16, 32, 64, 128):
        prompt, heads = 64 * sweep, 8
        line = [rides(b, heads, prompt, head_dim, hidden, rank) for b in range(1, 14336 // (sweep * heads) + 1)]
        assert line == sorted(line, reverse=True)
        most = sum(line) * sweep * heads
        assert most + sweep * heads > last                 # (to a batch of this length)
        last = most
