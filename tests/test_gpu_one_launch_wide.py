"""One launch per step with a unit's rows split over four waves and more than 128 rows (GPU, against the oracle, and
bit for bit against the two halves as launches of their own).  Tolerances: tests/harness.py."""
import numpy as np
import pytest
import torch

from paper_2402_09398_amd import binding
from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


def shape(**kw):
    d = dict(name="split-4-waves-wide", batch=50, heads=8, head_dim=128, prompt=300, steps=8, n_heavy=64, n_recent=64,
             rank=8, hidden=64, dtype="f16")
    d.update(kw)
    return wl.WORKLOADS[2].scaled(**d)


@pytest.mark.parametrize("w", [
    shape(), shape(n_heavy=128, n_recent=128), shape(n_heavy=255, n_recent=256, prompt=530, steps=4),
    shape(batch=40, heads=10, n_heavy=100, n_recent=60, rank=5, hidden=96), shape(prompt=140, steps=30, n_heavy=80, n_recent=80),
], ids=lambda w: f"{w.batch}x{w.heads}-{w.capacity}-{w.prompt}")
def test_against_oracle(w):
    gpu = hz.make_gpu(w)
    assert binding.lessdec_step_launches(gpu.desc) == 1
    del gpu
    rep = hz.run_workload(w, [0, 1, 7, 8, w.units // 2, w.units - 1])
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]


def test_same_bits_as_two_launches():
    w = shape(steps=6)
    inp = wl.all_inputs(w)
    q, k, v = (torch.from_numpy(inp[n]).cuda() for n in "qkv")
    got = []
    for halves in (False, True):
        gpu = hz.make_gpu(w)
        gpu.prefill(*(torch.from_numpy(inp[n]).cuda() for n in "QKV"))
        outs = torch.empty_like(q)
        for t in range(w.steps):
            if halves:
                gpu.step_features(q[t], k[t])
                gpu.step_attend(q[t], k[t], v[t], outs[t])
            else:
                gpu.step(q[t], k[t], v[t], outs[t])
        gpu.state_sync()
        torch.cuda.synchronize()
        got.append([x.cpu().numpy().copy() for x in (outs, gpu.acc, gpu.H, gpu.z, gpu.pos, gpu.psi)])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
