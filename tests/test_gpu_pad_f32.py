"""A factors of 3x3 convolutions from zero-padded fp32 planes: image sizes that put the groups of four at every place of a padded
row (a group may run into the next row or the next plane), one plane and several, against the patch matrix in float64."""
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C", [(1, 1), (3, 5)])
@pytest.mark.parametrize("h,w", [(5, 5), (5, 7), (6, 9), (7, 7), (8, 13), (9, 11), (12, 10), (14, 14), (15, 17), (31, 29), (33, 6)])
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
