"""Lambda-masking taken through the prompt, fp16 storage: the masked rows, whose scores come from digit planes (GPU).

Tolerances: tests/harness.py (against the oracle); values that are not finite: which outputs they may reach.
"""
import numpy as np
import pytest

from paper_2402_09398_amd import workloads as wl
from tests import harness as hz
from tests.test_gpu_digits import shape

pytestmark = pytest.mark.gpu
FLAGS = 2 | 4                                            # Lambda-masking, active through the prompt


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("value", [np.inf, -np.inf])
@pytest.mark.parametrize("n_heavy,key", [(4, 20), (36, 50), (4, 70), (4, 93)])
def test_infinite_value(n_heavy, key, value, head_dim):
    """One value row holds an infinity.  Rows before it and other columns are those without it, bit for bit.  Rows that the
    pair reaches with a prefix state (whole blocks of 64 keys older than the windows of 16 queries) have that infinity for an
    output: no other tile of 32 keys adds a weight of zero times it, which is not a number."""
    w = shape(260, steps=0, n_heavy=n_heavy, n_recent=20, head_dim=head_dim)
    clean = wl.all_inputs(w)
    dirty = {k: v.copy() for k, v in clean.items()}
    dirty["V"][:, key, 7] = value
    a, b = (hz.gpu_run(w, x, flags=FLAGS)["prefill_out"] for x in (clean, dirty))
    same = a.view(np.uint16) == b.view(np.uint16)
    assert same[:, :, [c for c in range(head_dim) if c != 7]].all()
    assert same[:, :key // 16 * 16].all()                # (rows of the key's own 16 share its block)
    rows = [t for t in range(w.prompt) if (t // 16 * 16 - w.n_recent) // 64 * 64 > key]
    assert len(rows) > 50 and (b[:, rows, 7] == value).all()


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("which", ["K", "Q", "KQ"])
def test_values_without_digits(which, head_dim):
    """Elements of 127 and more: their tiles, and all tiles of a wave whose queries hold one, are multiplied in fp64."""
    w = shape(150, head_dim=head_dim, q_per_kv=2, n_heavy=5, n_recent=20)
    inp = wl.all_inputs(w)
    rng = np.random.default_rng(6)
    for name in which:
        x = inp[name].reshape(w.units, -1, w.prompt, head_dim)
        for value in (126.9375, -126.9375, 127.0, -300.0):
            for u in range(w.units):
                for head in range(x.shape[1]):
                    x[u, head, rng.integers(2, w.prompt), rng.integers(head_dim)] = value
    other = {"K": "Q", "Q": "K"}.get(which)              # what the large channel meets is small, so that the rows stay soft
    if other:
        big = np.abs(inp[which].astype(np.float32)).reshape(-1, head_dim).max(axis=0) > 100
        inp[other][..., big] *= np.float16(1 / 64)
    units = list(range(w.units))
    res = hz.gpu_run(w, inp, flags=FLAGS)
    rep = hz.check_against_oracle(w, inp, units, res, flags=FLAGS)
    rep.failures.extend(hz.check_every_unit(w, res, flags=FLAGS))
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]


def test_units_in_several_shares():
    """More tokens than the digits' part of the workspace holds (0.7 million of D = 128): the first, middle and last units as
    in a call of their own."""
    import torch
    batch, heads, p, d = 400, 32, 112, 128
    g = torch.Generator(device="cuda").manual_seed(3)
    full = {n: torch.randn(batch, heads, p, d, generator=g, device="cuda").half() for n in "QKV"}

    def prefill(x):
        gpu = hz.make_gpu(shape(p, batch=x["Q"].shape[0], heads=heads, n_recent=20), flags=FLAGS)
        out = torch.empty_like(x["Q"])
        gpu.prefill(x["Q"].contiguous(), x["K"].contiguous(), x["V"].contiguous(), out=out)
        torch.cuda.synchronize()
        return [t.reshape(x["Q"].shape[0], heads, *t.shape[1:]) if t.shape[0] != x["Q"].shape[0] else t
                for t in (out, gpu.acc, gpu.pos, gpu.H, gpu.z)]

    whole = prefill(full)
    for part in (slice(0, 3), slice(197, 203), slice(397, 400)):
        (out, acc, pos, H, z), (out1, acc1, pos1, H1, z1) = ([t[part] for t in whole], prefill({n: x[part] for n, x in full.items()}))
        assert torch.equal(out, out1) and torch.equal(pos, pos1) and torch.equal(H, H1) and torch.equal(z, z1)
        # column sums of at most p positive terms, which another number of units adds in another order
        assert torch.allclose(acc, acc1, rtol=p * 2.0 ** -53, atol=0)
