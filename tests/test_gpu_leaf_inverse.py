"""The one-workgroup inverse at the edges of its 32-row blocks, size classes and tile deals, against numpy in float64, and the
pivot it names when a matrix is not positive definite."""
import numpy as np
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 31, 32, 33, 63, 65, 96, 127, 129, 160, 161, 191, 193, 224, 225, 255, 257, 287, 288]


def _invert(A, G, gamma):
    layers = [wl.fc_layer(4, A.shape[0], G.shape[0], 0)]
    ctx = kfac.Context(layers)
    dA, dG = torch.from_numpy(A).cuda(), torch.from_numpy(G).cuda()
    Ai, Gi = torch.full_like(dA, 3.0), torch.full_like(dG, 3.0)
    pi, info = torch.zeros(1, device="cuda"), torch.full((2,), -1, dtype=torch.int32, device="cuda")
    kfac.kfac_invert(ctx, layers, [dA], [dG], gamma, [Ai], [Gi], pi, info)
    torch.cuda.synchronize()
    ctx.close()
    return Ai.cpu().numpy(), Gi.cpu().numpy(), float(pi), info.tolist()


@pytest.mark.parametrize("n", SIZES)
def test_inverse(n):
    rng = np.random.default_rng(n)
    X = []
    for scale in (1.0, 1e-6):
        b = rng.standard_normal((2 * n + 8, n))
        s = np.exp(rng.uniform(-2, 2, n))          # rows of different magnitude
        x = (b.T @ b / len(b) * s[:, None] * s[None, :] * scale).astype(np.float32)
        X.append(np.ascontiguousarray((x + x.T) / np.float32(2)))
    Ai, Gi, pi, info = _invert(X[0], X[1], 1e-3)
    assert info == [0, 0]
    for x, got, damp in ((X[0], Ai, pi * 1e-3), (X[1], Gi, 1e-3 / pi)):
        d = x.astype(np.float64) + damp * np.eye(n)
        ref = np.linalg.inv(d)
        s = 1 / np.sqrt(np.diag(d))
        kappa = np.linalg.cond(d * s[:, None] * s[None, :])     # of the unit-diagonal matrix the kernel eliminates
        assert np.array_equal(got, got.T)
        # element-wise in the unit-diagonal scale: n kappa 2^-24 of the largest element there for the elimination, and
        # eight roundings (kappa 2^-24 each) outside it: pi, the damping and its sum, the scales, scaling and its undoing
        err = np.abs(got - ref) / s[:, None] / s[None, :]
        assert err.max() <= (n + 8) * kappa * 2.0 ** -24 * (np.abs(ref) / s[:, None] / s[None, :]).max() + 1e-12


@pytest.mark.parametrize("n,bad", [(1, 0), (32, 0), (32, 1), (33, 32), (100, 6), (100, 7), (160, 159), (224, 101), (288, 8), (288, 271), (288, 287)])
def test_first_non_positive_pivot(n, bad):
    rng = np.random.default_rng(n + bad)
    b = rng.standard_normal((2 * n + 8, n))
    x = (b.T @ b / len(b)).astype(np.float32)
    x = np.ascontiguousarray((x + x.T) / np.float32(2))
    x[bad, bad] = -1.0
    _, _, _, info = _invert(x, np.eye(4, dtype=np.float32), 0.0)
    assert info == [bad + 1, 0]


def _parallel_pairs(rng, n, rho):
    """Second moments of variables whose neighbours 2 m and 2 m + 1 are correlated by rho."""
    x = rng.standard_normal((4 * n, n))
    second = x[:, 1::2]
    second[:] = rho * x[:, 0:2 * (n // 2):2] + np.sqrt(1 - rho * rho) * second
    return x.T @ x / len(x)


def _smooth_patches(rng, channels, k, damp):
    """Second moments of the k x k patches of smooth images."""
    hw, f = 28, np.fft.fftfreq(28)
    cols = []
    for _ in range(8):
        spectrum = np.fft.fft2(rng.standard_normal((channels, hw, hw))) / (0.002 + f[:, None] ** 2 + f[None, :] ** 2)
        image = np.fft.ifft2(spectrum).real
        image = np.maximum(image / image.std(), 0.0)
        image = np.pad(image, ((0, 0), (k // 2, k // 2), (k // 2, k // 2)))
        cols.append([image[c, y:y + hw, x:x + hw].ravel() for c in range(channels) for y in range(k) for x in range(k)])
    m = np.concatenate(cols, axis=1)
    return m @ m.T / m.shape[1] + damp * np.eye(len(m))


# one tile (whole and with a remainder); several; all of a leaf; leaves behind products (577: 288 and 289, which is 160 and 129)
@pytest.mark.parametrize("kind,n,value", [("pairs", n, rho) for n in (31, 32) for rho in (0.995, 0.9995, 0.99995)] +
                         [("pairs", n, 0.995) for n in (70, 288, 577)] + [("chain", 32, 0.9999), ("patches", (3, 7), 1e-2),
                          ("patches", (3, 7), 1e-3), ("patches", (32, 3), 1e-2), ("patches", (50, 3), 1e-3)])
def test_correlated_neighbours(kind, n, value):
    """Neighbouring taps of a patch (and gamma_i, beta_i of a BatchNorm layer) are strongly correlated variables: the rows
    of two successive pivots are nearly parallel, and the second pivot is small beside the first."""
    rng = np.random.default_rng(7)
    if kind == "pairs":
        x = _parallel_pairs(rng, n, value)
    elif kind == "chain":
        x = value ** np.abs(np.arange(n)[:, None] - np.arange(n)[None, :])
    else:
        x = _smooth_patches(rng, n[0], n[1], value)
    x = x.astype(np.float32)
    x = np.ascontiguousarray((x + x.T) / np.float32(2))
    got, _, _, info = _invert(x, np.eye(4, dtype=np.float32), 0.0)
    assert info == [0, 0]
    d = x.astype(np.float64)
    s = 1 / np.sqrt(np.diag(d))
    kappa = np.linalg.cond(d * s[:, None] * s[None, :])
    scaled = (1 / s)[:, None] * (1 / s)[None, :]
    ref = np.linalg.inv(d) * scaled
    # An elimination in fp32 that takes the pivots one after the other stays below 1.1 kappa 2^-24 of the largest element on
    # one tile (30 draws of every rho), and below 2.1 on these larger ones, whose products carry 2^-23 each: twice the latter.
    assert np.abs(got * scaled - ref).max() <= 4 * kappa * 2.0 ** -24 * np.abs(ref).max()


def _eliminate(x):
    """The inverse by an elimination in fp32 of the unit-diagonal matrix, one pivot after the other."""
    n, s = len(x), 1 / np.sqrt(np.diag(x))
    t = -x * s[:, None] * s[None, :]
    for p in range(n):
        u = t[p].copy()
        q = np.float32(-1) / u[p]
        u[p] += np.float32(1)
        t += (q * u)[:, None] * u[None, :]
    t[np.arange(n), np.arange(n)] += np.float32(2)
    assert t.dtype == np.float32
    return t * s[:, None] * s[None, :]


# The mean over the draws, in units of that elimination's error: 1.90, 1.28, 1.09, 0.88.  Products of three bf16 planes, all 24 bits of
# the operands, give 2.04, 1.42, 1.53, 1.49: a tenth above that is the limit; without the product of the low planes it is 5.8, 3.7, 2.3, 1.8.
@pytest.mark.parametrize("kind,n,limit", [("pairs", 160, 2.25), ("pairs", 288, 1.56), ("patches", 160, 1.68), ("patches", 288, 1.64)])
def test_precision_where_rows_are_nearly_parallel(kind, n, limit):
    """The split of the operands costs nothing that the sums would not cost anyway."""
    ratio = []
    for seed in range(8):
        rng = np.random.default_rng(1000 * n + seed)
        x = (_parallel_pairs(rng, n, 0.9995) if kind == "pairs" else _smooth_patches(rng, n // 9, 3, 1e-3)).astype(np.float32)
        x = np.ascontiguousarray((x + x.T) / np.float32(2))
        got, _, _, info = _invert(x, np.eye(4, dtype=np.float32), 0.0)
        assert info == [0, 0]
        d = x.astype(np.float64)
        s = np.sqrt(np.diag(d))
        ref = np.linalg.inv(d) * s[:, None] * s[None, :]
        err = [np.linalg.norm(y * s[:, None] * s[None, :] - ref) for y in (got, _eliminate(x))]
        ratio.append(err[0] / err[1])
    print(kind, n, np.mean(ratio))
    assert np.mean(ratio) <= limit


@pytest.mark.parametrize("n", [64, 65, 96, 128, 160, 200, 256, 288])
@pytest.mark.parametrize("kind", ["diagonal", "steep", "far"])
def test_blocks_of_different_magnitude(n, kind):
    """Panel blocks are scaled one by one: zero blocks, blocks whose elements grow large once their rows are swept beside others
    that stay small, and couplings far below the diagonal."""
    rng = np.random.default_rng(n)
    b = rng.standard_normal((2 * n + 8, n))
    x = b.T @ b / len(b)
    block = np.arange(n) // 32
    if kind == "diagonal":
        x = np.where(block[:, None] == block[None, :], x, 0.0)
    elif kind == "steep":      # the first block nearly singular, the others tied to it
        first = block == 0
        q, _ = np.linalg.qr(rng.standard_normal((32, 32)))
        x[np.ix_(first, first)] = q @ np.diag(np.geomspace(1, 1e-3, 32)) @ q.T
        x[np.ix_(first, ~first)] *= 1e-3
        x[np.ix_(~first, first)] *= 1e-3
    else:
        x = np.where(block[:, None] == block[None, :], x, x * 2.0 ** -18)
    x = x.astype(np.float32)
    x = np.ascontiguousarray((x + x.T) / np.float32(2))
    got, _, _, info = _invert(x, np.eye(4, dtype=np.float32), 0.0)
    assert info == [0, 0]
    d = x.astype(np.float64)
    s = 1 / np.sqrt(np.diag(d))
    kappa = np.linalg.cond(d * s[:, None] * s[None, :])
    scaled = (1 / s)[:, None] * (1 / s)[None, :]
    ref = np.linalg.inv(d) * scaled
    # the bound of test_correlated_neighbours; where blocks do not touch, each is as accurate as if it were alone, to what its
    # scale keeps of elements 2^-18 of the largest (2^-22 of them)
    err = np.abs(got * scaled - ref)
    assert err.max() <= 4 * kappa * 2.0 ** -24 * np.abs(ref).max()
    if kind == "diagonal":
        assert not err[block[:, None] != block[None, :]].any()
    if kind == "far":
        off = block[:, None] != block[None, :]
        assert err[off].max() <= 4 * n * kappa * 2.0 ** -22 * np.abs(ref[off]).max()


def test_leaves_of_all_sizes_in_one_call():
    """One launch takes the leaves of all sizes: the same bits as a call per size."""
    X = {}
    for n in SIZES:
        rng = np.random.default_rng(n)
        b = rng.standard_normal((2 * n + 8, n))
        x = (b.T @ b / len(b)).astype(np.float32)
        X[n] = np.ascontiguousarray((x + x.T) / np.float32(2))
    layers = [wl.fc_layer(4, n, n, 0) for n in SIZES]
    ctx = kfac.Context(layers)
    A = [torch.from_numpy(X[n]).cuda() for n in SIZES]
    Ai, Gi = [torch.zeros_like(a) for a in A], [torch.zeros_like(a) for a in A]
    pi, info = torch.zeros(len(SIZES), device="cuda"), torch.full((2 * len(SIZES),), -1, dtype=torch.int32, device="cuda")
    kfac.kfac_invert(ctx, layers, A, A, 1e-3, Ai, Gi, pi, info)
    torch.cuda.synchronize()
    ctx.close()
    assert not info.any()
    for q, n in enumerate(SIZES):
        one = _invert(X[n], X[n], 1e-3)
        assert np.array_equal(Ai[q].cpu().numpy(), one[0]) and np.array_equal(Gi[q].cpu().numpy(), one[1]), n
