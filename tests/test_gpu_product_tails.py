"""Launches of 128-row tiles with a few tiles more than the chip holds at once: the contractions of those last tiles are split
and added up by a second kernel.  U = G^-1 dW A^-1 of several layers against float64 products.  With the fp32 instruction
also long products of few 64-row tiles."""
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


def _precondition(layers, opts=None):
    """(the profile's entries of one kfac_precondition) after a check of the results."""
    gen = torch.Generator(device="cuda").manual_seed(layers[0].dA)
    G = [torch.randn(L.dG, L.dG, device="cuda", generator=gen) for L in layers]
    A = [torch.randn(L.dA, L.dA, device="cuda", generator=gen) for L in layers]
    W = [torch.randn(L.dG, L.dA, device="cuda", generator=gen) for L in layers]
    for x in G + A:
        x.copy_((x + x.t()) * 0.5)
    ctx = kfac.Context(layers, opts=opts)
    out = [torch.full((L.dG * L.dA + 64,), 7.25, device="cuda") for L in layers]
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_precondition(ctx, layers, G, A, W, out)
    torch.cuda.synchronize()
    entries = kfac.kfac_profile_read(ctx)
    for L, g, a, w, u in zip(layers, G, A, W, out):
        assert bool((u[L.dG * L.dA:] == 7.25).all())
        g, a, w = g.double(), a.double(), w.double()
        # every product carries 2^-23, a sum of K terms K 2^-24 of the sum of magnitudes at most; two contractions follow each other
        bound = (L.dA + L.dG + 8) * 2.0 ** -23 * (g.abs() @ w.abs() @ a.abs())
        assert bool(((u[:L.dG * L.dA].view(L.dG, L.dA) - g @ w @ a).abs() <= bound).all())
    ctx.close()
    return entries


# tiles of either product: 7 * 81 = 512 + 55 (the split tiles belong to one layer), 8 * 81 = 512 + 136 (to two), ragged K
@pytest.mark.parametrize("n,d", [(7, 1100), (8, 1085)])
def test_precondition_with_split_tails(n, d):
    entries = _precondition([wl.fc_layer(4, d, d, 0)] * n)
    assert [e["kernel"] for e in entries].count("gemm_reduce") == 2


# 48 tiles in four parts beside 12 in two and a whole one (50 rows); as many parts as there may be
@pytest.mark.parametrize("sizes", [[(1501, 77), (333, 70), (50, 50)], [(4096, 10)]])
def test_long_products_of_few_tiles_with_the_fp32_instruction(sizes):
    entries = _precondition([wl.fc_layer(4, d, e, 0) for d, e in sizes], kfac.options(fp32_products=kfac.KFAC_PRODUCTS_FP32_MFMA))
    first, second = entries[:2]
    assert (first["kernel"], first["variant"], second["kernel"]) == ("gemm_f32", 1, "gemm_reduce")
    tiles = -(-sizes[0][0] // 64) * -(-sizes[0][1] // 64)
    assert first["workgroups"] >= 2 * tiles
