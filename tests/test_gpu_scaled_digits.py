"""Row pass of the prompt phase with fp16 storage: rows scaled by powers of two before they are split into digits, lowest
digit planes left out where they are empty, units taking turns in the digits' workspace (GPU).

Tolerances: tests/harness.py (against the oracle), bit for bit where the same units run in another share.
"""
import numpy as np
import pytest

from paper_2402_09398_amd import workloads as wl
from tests import harness as hz
from tests.test_gpu_digits import run, shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("kind", ["scales", "halves-of-the-block", "wide", "zero", "edge"])
def test_scales_and_lowest_digits(kind, head_dim):
    w = shape(100, head_dim=head_dim, q_per_kv=2)
    inp = wl.all_inputs(w)
    rng = np.random.default_rng(11)
    K, Q = inp["K"], inp["Q"]
    if kind == "scales":                                 # every row another scale, down to subnormals
        K *= np.float16(2.0) ** -rng.integers(0, 15, K.shape[:-1] + (1,)).astype(np.float16)
        Q *= np.float16(2.0) ** -rng.integers(0, 4, Q.shape[:-1] + (1,)).astype(np.float16)
    elif kind == "halves-of-the-block":                  # lowest digits in one 64-wide block only, in K or in Q or in both
        for x, part in ((K, 0), (Q, head_dim // 2)):
            x[..., 30:60, part + 3] = np.float16(2.0 ** -24) * rng.integers(1, 1024, x[..., 30:60, 0].shape)
    elif kind == "wide":                                 # all four digits in use: 126.9 beside the smallest halves
        K[..., 5::7, 1] = np.float16(126.9375)
        Q[..., 1] = np.float16(2.0 ** -24) * rng.integers(-1000, 1000, Q.shape[:-1])
        Q[..., 9::11, 2] = np.float16(-126.9375)
        K[..., 2] = np.float16(2.0 ** -23)
    elif kind == "zero":
        K[..., 16:48, :] = 0
        Q[..., 20:40, :] = 0
    else:                                                # largest values just below and at 127 / 64 of a power of two
        for i, v in enumerate((1.984375, 1.9833984375, 3.96875, 3.966796875, 0.9921875, 1.0, 1.9990234375)):
            K[..., i::7, 0] = np.float16(v)
            Q[..., i::7, 0] = np.float16(v)
    run(w, inp)


def test_units_in_several_shares():
    """More tokens than the digits' part of the workspace holds (0.7 million of D = 128): the first and the last units
    as in a call of their own."""
    import torch
    batch, heads, p, d = 400, 32, 112, 128
    g = torch.Generator(device="cuda").manual_seed(2)
    full = {n: torch.randn(batch, heads, p, d, generator=g, device="cuda").half() for n in "QKV"}

    def prefill(x):
        gpu = hz.make_gpu(shape(p, batch=x["Q"].shape[0], heads=heads))
        out = torch.empty_like(x["Q"])
        gpu.prefill(x["Q"].contiguous(), x["K"].contiguous(), x["V"].contiguous(), out=out)
        torch.cuda.synchronize()
        return [t.reshape(x["Q"].shape[0], heads, *t.shape[1:]) if t.dim() < 4 else t for t in (out, gpu.acc, gpu.pos)]

    whole = prefill(full)
    for part in (slice(0, 3), slice(197, 203), slice(397, 400)):
        (out, acc, pos), (out1, acc1, pos1) = ([t[part] for t in whole], prefill({n: x[part] for n, x in full.items()}))
        assert torch.equal(out, out1) and torch.equal(pos, pos1)
        # column sums of at most p positive terms, which another number of units adds in another order
        assert torch.allclose(acc, acc1, rtol=p * 2.0 ** -53, atol=0)
