"""Launches of 128-row tiles with a few tiles more than the chip holds at once: the contractions of those last tiles are split
and added up by a second kernel.  U = G^-1 dW A^-1 of several layers against float64 products."""
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


# tiles of either product: 7 * 81 = 512 + 55 (the split tiles belong to one layer), 8 * 81 = 512 + 136 (to two), ragged K
@pytest.mark.parametrize("n,d", [(7, 1100), (8, 1085)])
def test_precondition_with_split_tails(n, d):
    layers = [wl.fc_layer(4, d, d, 0)] * n
    gen = torch.Generator(device="cuda").manual_seed(d)
    G, A, W = [[torch.randn(d, d, device="cuda", generator=gen) for _ in layers] for _ in range(3)]
    for x in G + A:
        x.copy_((x + x.t()) * 0.5)
    ctx = kfac.Context(layers)
    out = [torch.full((d * d + 64,), 7.25, device="cuda") for _ in layers]
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_precondition(ctx, layers, G, A, W, out)
    torch.cuda.synchronize()
    assert [e["kernel"] for e in kfac.kfac_profile_read(ctx)].count("gemm_reduce") == 2
    for g, a, w, u in zip(G, A, W, out):
        assert bool((u[d * d:] == 7.25).all())
        g, a, w = g.double(), a.double(), w.double()
        # every product carries 2^-23, a sum of K terms K 2^-24 of the sum of magnitudes at most; two contractions follow each other
        bound = (2 * d + 8) * 2.0 ** -23 * (g.abs() @ w.abs() @ a.abs())
        assert bool(((u[:d * d].view(d, d) - g @ w @ a).abs() <= bound).all())
    ctx.close()
