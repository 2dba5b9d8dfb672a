"""Bias borders of factors whose long contraction is split into many parts: the row sums of the parts are added up by the
reduction, for factors of one and of several tiles, with and without a running average."""
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


# parts: 7 (slabs of 32 rows), 33 and 98 (slabs of 8 rows); 49 = one tile, 147 = three rows of tiles, the last of them 19 rows
@pytest.mark.parametrize("N,size", [(2, 224), (10, 224), (31, 226)])
@pytest.mark.parametrize("c", [1, 3])
@pytest.mark.parametrize("dtype", [kfac.KFAC_F32, kfac.KFAC_BF16])
def test_border_of_many_parts(N, size, c, dtype):
    L = wl.Layer(N, c, 64, 7, 2, 3, size, size, 1)
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randn(N, c, size, size, device="cuda", generator=gen).clamp_(min=0)
    if dtype == kfac.KFAC_BF16:
        x = x.bfloat16()
    A = torch.randn(L.dA, L.dA, device="cuda", generator=gen)
    A = (A + A.t()).contiguous()
    A0 = A.double()
    ctx = kfac.Context([L], dtype)
    kfac.kfac_stats(ctx, [L], dtype, [x], None, 0.75, True, [A], [torch.empty(64, 64, device="cuda")])
    torch.cuda.synchronize()
    ctx.close()
    m = torch.nn.functional.unfold(x.double(), 7, padding=3, stride=2).permute(1, 0, 2).reshape(49 * c, -1)
    m = torch.cat([m, torch.ones(1, m.shape[1], device="cuda", dtype=torch.float64)])
    ref = 0.75 * A0 + 0.25 * (m @ m.t()) / m.shape[1]
    # parts of at most 4096 terms, sums of at most 128 parts and three roundings of the running average
    bound = (4096 + 128) * 2.0 ** -24 * 0.25 * (m @ m.t()) / m.shape[1] + 2.0 ** -22 * A0.abs()
    assert bool(((A.double() - ref).abs() <= bound).all())
    assert bool((A == A.t()).all())
