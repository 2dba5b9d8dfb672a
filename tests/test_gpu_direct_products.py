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


@pytest.mark.parametrize("d,d_out,variant", [(256, 32, 2), (576, 64, 2), (1023, 833, 3)])
def test_sums_that_cancel_across_steps(d, d_out, variant):
    """W A^-1 where what one 16-wide step adds is taken away by the next, as in products with the inverse of a factor whose
    neighbouring variables are correlated: the sums of the steps of one wavefront are far larger than the result."""
    L = wl.fc_layer(4, d, d_out, 0)
    gen = torch.Generator(device="cuda").manual_seed(d)
    A = torch.randn(d, d, device="cuda", generator=gen)
    W = torch.zeros(d_out, d, device="cuda")
    edges = torch.arange(16, d, 16, device="cuda")
    W[:, edges - 1] = torch.randn(d_out, len(edges), device="cuda", generator=gen)
    W[:, edges] = -W[:, edges - 1]
    A[:, edges] = A[:, edges - 1] * (1 + 2.0 ** -12 * torch.randn(d, len(edges), device="cuda", generator=gen))
    out = torch.empty(d_out, d, device="cuda")
    ctx = kfac.Context([L])
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_precondition(ctx, [L], [torch.eye(d_out, device="cuda")], [A], [W], [out])
    torch.cuda.synchronize()
    assert variant in {e["variant"] for e in kfac.kfac_profile_read(ctx)}
    ctx.close()
    W, A = W.double(), A.double()
    steps = -(-d // 16)
    step = (W ** 2 @ (A ** 2).t() / steps).sqrt()   # what a step adds
    # A wavefront rounds its sum of m steps, sqrt(m) of that, once a step for m = 1 .. M; then come four sums of the planes'
    # low-order terms and three of the wavefronts.  A rounding is 2^-24 / sqrt(3) at most, uniform in half a unit.  (Six
    # roundings a step, or ones that do not go to nearest, are outside: 6.8 for d = 256, where this is 4.8.)
    M = steps / 4
    rms = ((out.double() - W @ A.t()) / (step * 2.0 ** -24)).pow(2).mean().sqrt()
    assert float(rms) <= ((2 * M * (M + 1) + 7 * M) / 3) ** 0.5


@pytest.mark.parametrize("sizes", [[(1879, 1382)], [(2574, 1056), (427, 1047), (134, 214)], [(1000, 512)] * 6])
def test_error_of_middle_sizes(sizes):
    """Gradients of middle size keep the direct kernels' error, though a staged one would be the faster by up to 1.5."""
    layers = [wl.fc_layer(4, d_in, d_out, 0) for d_in, d_out in sizes]
    gen = torch.Generator(device="cuda").manual_seed(len(sizes))

    def inverse(d):
        x = torch.randn(d, d, device="cuda", generator=gen) * (0.6 / d ** 0.5)
        return (x + x.t() + 1.5 * torch.eye(d, device="cuda")).contiguous()

    A, G = [inverse(L.dA) for L in layers], [inverse(L.dG) for L in layers]
    W = [torch.randn(L.dG, L.dA, device="cuda", generator=gen) for L in layers]
    U = [torch.empty_like(w) for w in W]
    ctx = kfac.Context(layers)
    kfac.kfac_precondition(ctx, layers, G, A, W, U)
    torch.cuda.synchronize()
    ctx.close()
    for L, a, g, w, u in zip(layers, A, G, W, U):
        ref = g.double() @ w.double() @ a.double()
        # a wavefront rounds its sum of m = 1 .. K / 64 steps once each, 2^-24 / sqrt(3) of it at most: sqrt(K / 64 / 6) 2^-24 of the
        # result, and two sums of partial ones per contraction; half as much again for what is not random
        bound = 1.5 * 2.0 ** -24 * ((L.dA + L.dG) / 64 / 6 + 2) ** 0.5
        assert float((u.double() - ref).norm() / ref.norm()) <= bound
