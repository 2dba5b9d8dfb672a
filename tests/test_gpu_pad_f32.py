"""A factors of 3x3 convolutions from zero-padded fp32 planes: image sizes that put the groups of four at every place of a padded
row (a group may run into the next row or the next plane), one plane and several, against the patch matrix in float64."""
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


# from 254x254 on, a padded plane has 65536 positions and more: divisions instead of reciprocals
@pytest.mark.parametrize("N,C", [(1, 1), (3, 5)])
@pytest.mark.parametrize("h,w", [(254, 254), (300, 259), (8, 33000), (5, 5), (5, 7), (6, 9), (7, 7), (8, 13), (9, 11), (12, 10), (14, 14), (15, 17), (31, 29), (33, 6)])
def test_factor_of_padded_planes(N, C, h, w):
    L = wl.Layer(N, C, 4, 3, 1, 1, h, w, 1)
    gen = torch.Generator(device="cuda").manual_seed(100 * h + w)
    x = torch.randn(N, C, h, w, device="cuda", generator=gen)
    A = torch.full((L.dA, L.dA), float("nan"), device="cuda")
    ctx = kfac.Context([L])
    kfac.kfac_stats(ctx, [L], kfac.KFAC_F32, [x], None, 0.0, True, [A], [torch.empty(4, 4, device="cuda")])
    torch.cuda.synchronize()
    ctx.close()
    m = torch.nn.functional.unfold(x.double(), 3, padding=1).permute(1, 0, 2).reshape(9 * C, -1)
    m = torch.cat([m, torch.ones(1, m.shape[1], device="cuda", dtype=torch.float64)])
    # the whole correlation less up to two lines plus a corner: each sum has at most N (h + 5) (w + 5) terms of this size
    terms = N * (h + 5) * (w + 5)
    bound = 4 * (terms + 16) * 2.0 ** -24 * float((m.abs() @ m.abs().t()).max()) / m.shape[1]
    assert float((A.double() - m @ m.t() / m.shape[1]).abs().max()) <= bound


def test_more_positions_than_32_bits():
    """2^31 positions and more (divisions in 64 bits): the blocks of the first and the last channel."""
    C, size = 129, 4095
    L = wl.Layer(1, C, 4, 3, 1, 1, size, size, 0)
    assert C * (size + 2) ** 2 > 2 ** 31
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(1, C, size, size, device="cuda", generator=gen)
    A = torch.empty(L.dA, L.dA, device="cuda")
    ctx = kfac.Context([L])
    kfac.kfac_stats(ctx, [L], kfac.KFAC_F32, [x], None, 0.0, True, [A], [torch.empty(4, 4, device="cuda")])
    torch.cuda.synchronize()
    ctx.close()
    m = torch.cat([torch.nn.functional.unfold(x[:, c:c + 1].double(), 3, padding=1)[0] for c in (0, C - 1)])
    ref = (m @ m.t()) / m.shape[1]
    rows = torch.tensor(list(range(9)) + list(range(L.dA - 9, L.dA)), device="cuda")
    # parts of at most 4096 terms and sums of at most 4100 parts, each with errors of random sign: far below the sums' own bound
    assert float((A[rows][:, rows].double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
