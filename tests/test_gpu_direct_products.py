"""Small products (the direct kernels): U = G^-1 dW A^-1 of fully-connected layers whose sizes sit on the edges of their
32-row and 64-row tiles, the 16-wide steps and the four wavefronts that share a contraction, against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


def _symmetric(rng, n):
    x = rng.standard_normal((n, n)).astype(np.float32)
    return np.ascontiguousarray((x + x.T) * np.float32(0.5))


# variant 2: 32 x 32 tiles, 3: 64 x 64
@pytest.mark.parametrize("d_in,d_out,variant", [(d_in, d_out, 2) for d_in, d_out in (
    (1, 1), (3, 2), (15, 17), (16, 16), (31, 33), (32, 64), (63, 65), (64, 15), (79, 96), (129, 31), (255, 257), (576, 64),
    (1023, 12))] + [(737, 641, 3), (720, 705, 3), (767, 703, 3)])
@pytest.mark.parametrize("bias", [0, 1])
def test_precondition_at_tile_edges(d_in, d_out, variant, bias):
    layers = [wl.fc_layer(4, d_in, d_out, bias), wl.fc_layer(4, max(1, d_in // 2), d_out + 1, bias)]
    rng = np.random.default_rng(1000 * d_in + d_out + bias)
    G = [_symmetric(rng, L.dG) for L in layers]
    A = [_symmetric(rng, L.dA) for L in layers]
    W = [rng.standard_normal((L.dG, L.dA)).astype(np.float32) for L in layers]
    ctx = kfac.Context(layers)
    dev = [[torch.from_numpy(x).cuda() for x in xs] for xs in (G, A, W)]
    guard = 7.25   # elements behind every result, which must stay
    out = [torch.full((L.dG * L.dA + 64,), guard, device="cuda") for L in layers]
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_precondition(ctx, layers, *dev, out)
    torch.cuda.synchronize()
    assert {e["variant"] for e in kfac.kfac_profile_read(ctx)} == {variant}
    for i, L in enumerate(layers):
        got = out[i].cpu().numpy().astype(np.float64)
        assert np.all(got[L.dG * L.dA:] == guard)
        ref = oracle.kfac_precondition(G[i].astype(np.float64), A[i].astype(np.float64), W[i])
        # every product carries 2^-23, a sum of K terms K 2^-24 of the sum of magnitudes at most; two contractions follow each other
        bound = (L.dA + L.dG + 8) * 2.0 ** -23 * (np.abs(G[i]).astype(np.float64) @ np.abs(W[i]) @ np.abs(A[i]))
        assert np.all(np.abs(got[:L.dG * L.dA].reshape(L.dG, L.dA) - ref) <= bound)
    ctx.close()
