"""Prompt phase, fp16: psi of the keys in the row pass's launch or in one of its own, on both sides of the other lines of the rule, and in a launch
of the first of several shares of the keys (GPU).  The same bits, see tests/test_gpu_maps_ride.py."""
import pytest

from tests import harness as hz
from tests.maps_rule import rides
from tests.test_gpu_digits import shape
from tests.test_gpu_maps_ride import test_both_sides_of_the_line as both_sides

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,rank,hidden,heads,prompt,batches", [
    (128, 16, 512, 32, 64, (72, 73)),                    # one workgroup a sweep, the widest weights
    (128, 8, 512, 16, 520, (33, 34)),                    # sweeps of nine workgroups
    (128, 8, 256, 16, 2000, (19, 20)),                   # of 32, narrower weights
    (64, 8, 512, 32, 64, (208, 209)),
    (64, 8, 512, 16, 1000, (49, 50)),                    # the most workgroups
    (64, 8, 96, 32, 100, (163, 164)),                    # a width that does not stay in registers
])
def test_lines(head_dim, rank, hidden, heads, prompt, batches):
    both_sides(head_dim, rank, hidden, heads, prompt, batches)


def test_several_shares_of_keys():
    """More keys than the digits' part of the workspace holds (352 MiB at 512 bytes a key): all maps ride with the first share."""
    import torch
    heads, prompt, batches = 16, 1000, (40, 46)          # 640 000 keys, 736 000
    assert all(rides(b, heads, prompt, 128, 96, 4) for b in batches)
    assert heads * batches[0] * 1024 * 516 < 352 << 20 < heads * batches[1] * 1024 * 516
    g = torch.Generator(device="cuda").manual_seed(4)
    x = {n: torch.randn(max(batches), heads, prompt, 128, generator=g, device="cuda").half() for n in "QKV"}
    res = []
    for b in batches:
        gpu = hz.make_gpu(shape(prompt, batch=b, heads=heads, rank=4, hidden=96))
        q, k, v = (x[n][:b].contiguous() for n in "QKV")
        out = torch.empty_like(q)
        gpu.prefill(q, k, v, out=out)
        torch.cuda.synchronize()
        n = min(batches) * heads
        res.append([out.reshape(b * heads, -1)[:n], gpu.psi[:n], gpu.pos[:n], gpu.H[:n], gpu.z[:n]])
    for a, b in zip(*res):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
