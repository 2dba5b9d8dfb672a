"""Contraction operand of pointwise layers with planes below 64 positions: runs of 16 bytes that begin and end inside planes, rows
that are no whole number of runs, workgroups that end inside a row, tensors and rows off any alignment.  Exact."""
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tdt", [(kfac.KFAC_F32, torch.float32), (kfac.KFAC_BF16, torch.bfloat16)])
@pytest.mark.parametrize("h,w", [(1, 1), (1, 2), (1, 3), (2, 4), (7, 7), (9, 7)])
@pytest.mark.parametrize("n,c,pad", [(1, 1, 0), (2, 300, 1), (5, 33, 3), (32, 70, 0)])
def test_rows_of_tiny_planes(h, w, n, c, pad, dtype, tdt):
    L = wl.Layer(n, c, 4, 1, 1, 0, h, w, 0)
    M = n * h * w
    ld = M + pad
    gen = torch.Generator(device="cuda").manual_seed(M + c)
    store = torch.randn(n * c * h * w + 3, device="cuda", generator=gen).to(tdt)
    act = store[3:].view(n, c, h, w)
    out = torch.full((c * ld + 11,), 7.0, device="cuda", dtype=tdt)
    ctx = kfac.Context([L], dtype)
    kfac.kfac_im2col(ctx, L, dtype, act, out[1:1 + c * ld].view(c, ld), ld)
    torch.cuda.synchronize()
    ctx.close()
    want = torch.full_like(out, 7.0)
    want[1:1 + c * ld].view(c, ld)[:, :M] = act.transpose(0, 1).reshape(c, M)
    assert torch.equal(out, want)
