"""Prompt phase, fp16: psi of the keys in the row pass's launch or in one of its own (GPU).

Both evaluate a row by the same arithmetic in the same order, so a unit's psi, state and outputs are the same bits on either side of
the rule's line.
"""
import pytest

from tests import harness as hz
from tests.maps_rule import rides
from tests.test_gpu_digits import shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,rank,hidden,heads,prompt,batches", [
    (128, 4, 128, 8, 64, (224, 225)),                    # one workgroup a sweep
    (128, 8, 512, 16, 130, (86, 87)),                    # the widest weights, ragged rows
    (128, 12, 512, 8, 500, (57, 58)),                    # features with padding, sweeps of eight workgroups
    (64, 8, 256, 8, 70, (409, 410)),
])
def test_both_sides_of_the_line(head_dim, rank, hidden, heads, prompt, batches):
    import torch
    assert [rides(b, heads, prompt, head_dim, hidden, rank) for b in batches] == [True, False]
    g = torch.Generator(device="cuda").manual_seed(4)
    x = {n: torch.randn(max(batches), heads, prompt, head_dim, generator=g, device="cuda").half() for n in "QKV"}
    res = []
    for b in batches:
        gpu = hz.make_gpu(shape(prompt, batch=b, heads=heads, head_dim=head_dim, rank=rank, hidden=hidden))
        q, k, v = (x[n][:b].contiguous() for n in "QKV")
        out = torch.empty_like(q)
        gpu.prefill(q, k, v, out=out)
        torch.cuda.synchronize()
        n = min(batches) * heads
        res.append([out.reshape(b * heads, -1)[:n], gpu.psi[:n], gpu.pos[:n], gpu.H[:n], gpu.z[:n]])
    for a, b in zip(*res):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
