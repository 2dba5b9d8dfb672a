"""Correlation form of 3x3 layers with bf16 activations at the edges of the padded copies' windows: image widths around the
groups of 8, one plane, planes whose last row ends the tensor.  The activations are small whole numbers, so every sum is exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


# the correlation form takes 2 (h + 2) (w + 2, up to a multiple of 8) <= 5 h w
@pytest.mark.parametrize("h,w", [(6, 6), (3, 22), (21, 4), (9, 5), (15, 9), (7, 13), (14, 14), (8, 15), (28, 28)])
@pytest.mark.parametrize("n,c", [(1, 1), (3, 5)])
def test_factor_of_padded_images(h, w, n, c):
    L = wl.Layer(n, c, 4, 3, 1, 1, h, w, 1)
    rng = np.random.default_rng(h * w + n)
    act = rng.integers(0, 8, (n, c, h, w)).astype(np.float32)
    grad = rng.integers(-3, 4, (n, 4, h, w)).astype(np.float32)
    store = torch.full((act.size + 16,), float("nan"), device="cuda", dtype=torch.bfloat16)   # NaN on both sides of the tensor
    store[8:8 + act.size] = torch.from_numpy(act.ravel()).cuda().bfloat16()
    A, G = torch.empty(L.dA, L.dA, device="cuda"), torch.empty(L.dG, L.dG, device="cuda")
    ctx = kfac.Context([L], kfac.KFAC_BF16)
    kfac.kfac_stats(ctx, [L], kfac.KFAC_BF16, [store[8:8 + act.size].view(n, c, h, w)],
                    [torch.from_numpy(grad).cuda().bfloat16()], 0.0, False, [A], [G])
    torch.cuda.synchronize()
    ctx.close()
    ref = oracle.kfac_stats(tuple(L), act, grad, 0.0, False, None, None)
    for got, want in zip((A, G), ref):   # exact sums; the scale and its product are rounded
        want = np.asarray(want, dtype=np.float64)
        assert (np.abs(got.cpu().numpy() - want) <= 4 * 2.0 ** -24 * np.abs(want)).all()
