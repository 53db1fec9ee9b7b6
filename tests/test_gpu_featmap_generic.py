"""Feature maps of the general path (fp64 matrix tiles, hidden units spread over blocks): ranks around the
tile of 16, hidden widths with a ragged last tile, odd row counts, both storage types, phi through the step's output
and psi through the state (GPU, against the oracle).  Tolerances: tests/harness.py."""
import numpy as np
import pytest
import torch

from paper_2402_09398_amd import LessDec, pack_weights
from paper_2402_09398_amd import workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(rank=1, hidden=1), dict(rank=4, hidden=15), dict(rank=8, hidden=512), dict(rank=16, hidden=130),
    dict(rank=17, hidden=200), dict(rank=64, hidden=512), dict(rank=64, hidden=2048, batch=1, heads=2),
    dict(rank=8, hidden=512, batch=17, heads=2), dict(rank=5, hidden=257, head_dim=64, q_per_kv=3),
    dict(rank=33, hidden=96, dtype="f16"), dict(rank=8, hidden=100, dtype="f16", head_dim=64),
    dict(rank=3, hidden=64, batch=40, heads=30, prompt=10, steps=3),
], ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
def test_general_feature_maps(kw):
    d = dict(name="general-maps", batch=2, heads=3, head_dim=128, prompt=20, steps=6, n_heavy=4, n_recent=4, dtype="f32")
    d.update(kw)
    w = wl.WORKLOADS[2].scaled(**d)
    rep = hz.run_workload(w, range(min(w.units, 40)))
    print("\n" + rep.summary(), flush=True)
    assert rep.ok(), rep.failures[:10]


def test_infinite_weight_beside_the_padding():
    """A hidden width that leaves a tile of 16 ragged, the last unit's layer-2 weight infinite: psi is infinite where
    that unit's activation is positive, as without padding, and not a number elsewhere (-inf times the tail of 0)."""
    w = wl.WORKLOADS[2].scaled(name="infinite-weight", batch=1, heads=2, head_dim=64, prompt=8, steps=0, n_heavy=4,
                               n_recent=4, rank=1, hidden=15, dtype="f32")
    inp = wl.all_inputs(w)
    W = wl.head_weights(w)
    W["Wk2"][:, 14, 0] = np.inf
    hidden = np.einsum("upd,ud->up", inp["K"].astype(np.float64), W["Wk1"][:, :, 14].astype(np.float64))
    assert np.abs(hidden).min() > 1e-3 and (hidden > 0).any() and (hidden < 0).any()
    gpu = LessDec(w.batch, w.heads, w.head_dim, w.n_heavy, w.n_recent, w.rank, w.hidden, w.dtype, pack_weights(W),
                  max_prompt=w.prompt)
    gpu.prefill(*(torch.from_numpy(inp[n]).cuda() for n in "QKV"))
    psi = gpu.psi.cpu().numpy()[..., 0]
    assert np.array_equal(np.isinf(psi), hidden > 0) and np.array_equal(np.isnan(psi), hidden < 0)
