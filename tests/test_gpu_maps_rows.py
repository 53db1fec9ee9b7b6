"""psi of many prompt keys with the weights in registers (fp16), against float64: units of every length around the pieces of 16 and 32
rows that the kernel takes, a length of one, both widths of the output (rank up to 8 and above) and every hidden width of the form (GPU)."""
import pytest

from paper_2402_09398_amd import pack_weights, workloads as wl
from tests import harness as hz
from tests.test_gpu_digits import shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prompt,batch,heads,head_dim,rank,hidden", [
    (1, 1100, 2, 128, 8, 512), (2, 511, 2, 64, 9, 384), (15, 70, 3, 128, 16, 512), (17, 64, 2, 128, 1, 256),
    (31, 40, 2, 64, 8, 128), (33, 33, 5, 128, 5, 512), (777, 2, 2, 128, 11, 512),
])
def test_psi_of_every_kept_key(prompt, batch, heads, head_dim, rank, hidden):
    import torch
    g = torch.Generator(device="cuda").manual_seed(9)
    w = shape(prompt, batch=batch, heads=heads, head_dim=head_dim, rank=rank, hidden=hidden, n_heavy=prompt, n_recent=1)
    gpu = hz.make_gpu(w)
    q, k, v = (torch.randn(batch, heads, prompt, head_dim, generator=g, device="cuda").half() for _ in "qkv")
    gpu.prefill(q, k, v)
    torch.cuda.synchronize()
    gelu = lambda x: 0.5 * x * torch.erfc(x * (-0.5 ** 0.5))  # noqa: E731
    W = pack_weights(wl.head_weights(w), "cuda")
    weights = [W[n].double() for n in ("Wk1", "Wk2", "Wk3")]
    want = torch.empty(batch, heads, prompt, rank, dtype=torch.float64, device="cuda")
    for h in range(heads):
        x = gelu(gelu(k[:, h].double() @ weights[0][h].t().contiguous()) @ weights[1][h].t().contiguous())
        want[:, h] = (x @ weights[2][h].t().contiguous()).abs()
    got = gpu.psi.reshape(batch, heads, -1, rank)[:, :, :prompt].double()
    # fp32 sums of D, then R' products of values near 1, each a few units of 2^-24 in the norm, and the activations' 2.5e-7
    err = (got - want).abs().max() / want.abs().max()
    assert torch.isfinite(got).all() and err < 3e-6, float(err)
