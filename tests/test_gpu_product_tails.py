"""Launches of 128-row tiles with a few tiles more than the chip holds at once: the contractions of those last tiles are split
and added up by a second kernel.  U = G^-1 dW A^-1 of several layers against float64 products, and inverses by their residual.
With the fp32 instruction also long products of few 64-row tiles."""
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


# 12 matrices of 2323 = 1152 + 1171 rows: every product of the first partition (rectangular with a transposed copy, symmetric
# with the old values and with the part above the diagonal left out) has a split tail.  8 of 1361 = 672 + 689: the 64-row tiles
# of the direct kernel take all four, contractions of 672 and 689.
@pytest.mark.parametrize("n,d,variant,reductions", [(6, 2323, 0, 4), (4, 1361, 3, 0)])
def test_inversion_of_ragged_matrices(n, d, variant, reductions):
    layers = [wl.fc_layer(4, d, d, 0)] * n
    gen = torch.Generator(device="cuda").manual_seed(d)
    X = []
    for _ in range(2 * n):   # 2 I + E, the norm of E about 1/2
        e = torch.randn(d, d, device="cuda", generator=gen) * (0.18 / d ** 0.5)
        X.append(e + e.t() + 2 * torch.eye(d, device="cuda"))
    out = [torch.full((d * d + 64,), float("nan"), device="cuda") for _ in X]
    pi, info = torch.zeros(n, device="cuda"), torch.zeros(2 * n, dtype=torch.int32, device="cuda")
    ctx = kfac.Context(layers)
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_invert(ctx, layers, X[:n], X[n:], 0.0, out[:n], out[n:], pi, info)
    torch.cuda.synchronize()
    entries = kfac.kfac_profile_read(ctx)
    ctx.close()
    assert not info.any()
    assert variant in {e["variant"] for e in entries if e["kernel"] == "gemm_f32_split"}
    assert sum(e["kernel"] == "gemm_reduce" for e in entries) == reductions
    for x, y in zip(X, out):
        assert bool(y[d * d:].isnan().all())
        y = y[:d * d].view(d, d)
        assert bool((y == y.t()).all())
        x, y = x.double(), y.double()
        # The residual of a block inverse is at most the rounding of its products, as above, times |X| |X^-1| once for
        # the product and once for the inverse it was made with.
        p = x.abs() @ y.abs()
        r = (x @ y - torch.eye(d, device="cuda", dtype=torch.float64)).abs()
        assert bool((r <= (d + 8) * 2.0 ** -23 * (p @ p)).all())
