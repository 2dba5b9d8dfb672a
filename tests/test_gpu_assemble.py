"""Factors of 3x3 convolutions around 256 channels, from where the rows of A are dealt out by channel (eight channels at a time,
those left over in order), and around the 256 channels that a workgroup takes at a time."""
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c", [255, 256, 257, 263, 264, 513])
@pytest.mark.parametrize("decay", [0.0, 0.75])
@pytest.mark.parametrize("bias", [0, 1])
def test_rows(c, decay, bias):
    L = wl.Layer(16, c, 8, 3, 1, 1, 5, 6, bias)
    gen = torch.Generator(device="cuda").manual_seed(c)
    x = torch.randn(L.N, c, 5, 6, device="cuda", generator=gen).clamp_(min=0)
    A = torch.randn(L.dA, L.dA, device="cuda", generator=gen)
    A = (A + A.t()).contiguous()
    A0, G = A.double(), torch.empty(8, 8, device="cuda")
    ctx = kfac.Context([L])
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_stats(ctx, [L], kfac.KFAC_F32, [x], None, decay, True, [A], [G])
    torch.cuda.synchronize()
    assert any(e["kernel"] == "assemble" for e in kfac.kfac_profile_read(ctx))
    ctx.close()
    m = torch.nn.functional.unfold(x.double(), 3, padding=1).permute(1, 0, 2).reshape(9 * c, -1)
    if bias:
        m = torch.cat([m, torch.ones(1, m.shape[1], device="cuda", dtype=torch.float64)])
    ref = decay * A0 + (1 - decay) * (m @ m.t()) / m.shape[1]
    # sums of at most 16 x 56 terms, 2^-22 a product, an image's sums less those of its border lines and plus those of its corners
    # (three times the sum of an image at most), three roundings of the running average
    bound = 3 * (16 * 56 + 4) * 2.0 ** -24 * (1 - decay) * (m.abs() @ m.abs().t()) / m.shape[1] + 2.0 ** -22 * A0.abs()
    assert bool(((A.double() - ref).abs() <= bound).all())
    assert bool((A == A.t()).all())


@pytest.mark.parametrize("c", [255, 256, 257, 263, 264, 513])
@pytest.mark.parametrize("decay", [0.0, 0.75])
def test_whole_numbers(c, decay):
    """Sums that fp32 holds exactly: what is left are the roundings of the factor 1 / (N hw) and of the running average."""
    L = wl.Layer(16, c, 8, 3, 1, 1, 5, 6, 1)
    gen = torch.Generator(device="cuda").manual_seed(c)
    x = torch.randint(-7, 8, (L.N, c, 5, 6), device="cuda", generator=gen).float()
    A = torch.randn(L.dA, L.dA, device="cuda", generator=gen)
    A = (A + A.t()).contiguous()
    A0, G = A.double(), torch.empty(8, 8, device="cuda")
    ctx = kfac.Context([L])
    kfac.kfac_stats(ctx, [L], kfac.KFAC_F32, [x], None, decay, True, [A], [G])
    torch.cuda.synchronize()
    ctx.close()
    m = torch.nn.functional.unfold(x.double(), 3, padding=1).permute(1, 0, 2).reshape(9 * c, -1)
    m = torch.cat([m, torch.ones(1, m.shape[1], device="cuda", dtype=torch.float64)])
    new = (1 - decay) * (m @ m.t()) / m.shape[1]
    # the factor, its product with the sum, the product of the old value, their sum: a rounding each
    assert bool(((A.double() - decay * A0 - new).abs() <= 2.0 ** -22 * (new.abs() + decay * A0.abs())).all())
