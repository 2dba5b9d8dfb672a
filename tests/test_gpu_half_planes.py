"""fp32 products through two fp16 planes with a scale per operand row (the staged kernels): edges of tiles and K tiles, and what
happens where the range of fp16 does not cover a row.  Every product stays within what an fp32 sum of fp32 products loses."""
import numpy as np
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


def _precondition(G, A, W, tile):
    L = wl.fc_layer(4, A.shape[0], G.shape[0], 0)
    with kfac.default_options(force_tile=tile):
        ctx = kfac.Context([L])
    dev = [[torch.from_numpy(x).cuda()] for x in (G, A, W)]
    out = torch.full((L.dG * L.dA + 64,), 7.25, device="cuda")
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_precondition(ctx, [L], *dev, [out])
    torch.cuda.synchronize()
    assert {e["variant"] for e in kfac.kfac_profile_read(ctx) if e["kernel"] == "gemm_f32_split"} == {0 if tile == 128 else 1}
    ctx.close()
    got = out.cpu().numpy()
    assert np.all(got[L.dG * L.dA:] == 7.25)
    return got[:L.dG * L.dA].reshape(L.dG, L.dA).astype(np.float64)


def _check(G, A, W, tile):
    got = _precondition(G, A, W, tile)
    G, A, W = (x.astype(np.float64) for x in (G, A, W))
    ref = G @ W @ A.T
    # Roundings of random sign: sqrt(K) 2^-24 of the sum of magnitudes, for two contractions one after the other, and the largest of
    # some 10^5 at five times that.  (Without the low plane it is 2^12 times as much.)
    bound = 5 * (np.sqrt(len(A)) + np.sqrt(len(G)) + 1) * 2.0 ** -24 * (np.abs(G) @ np.abs(W) @ np.abs(A).T)
    assert np.all(np.abs(got - ref) <= bound)
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


def _sym(rng, n):
    x = rng.standard_normal((n, n)).astype(np.float32)
    return np.ascontiguousarray((x + x.T) * np.float32(0.5))


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("d_in,d_out", [(1, 1), (3, 2), (31, 33), (32, 64), (63, 65), (64, 96), (66, 127), (97, 128), (129, 31),
                                        (161, 130), (255, 257), (391, 100)])
def test_products_at_tile_edges(d_in, d_out, tile):
    rng = np.random.default_rng(1000 * d_in + d_out)
    err = _check(_sym(rng, d_out), _sym(rng, d_in), rng.standard_normal((d_out, d_in)).astype(np.float32), tile)
    assert err < 1e-6


@pytest.mark.parametrize("tile", [64, 128])
def test_rows_outside_the_range_of_fp16(tile):
    """Elements the scale was not taken from and that are too large for it (the workgroup repeats the tile), rows that are zero
    where they are sampled, rows of zeros, subnormal elements; the ends of the fp32 range."""
    rng = np.random.default_rng(tile)
    d_in, d_out = 520, 200
    G, A = _sym(rng, d_out), _sym(rng, d_in)
    W = rng.standard_normal((d_out, d_in)).astype(np.float32)
    W[3, 77] = 3e5                      # between the sampled chunks
    W[5, :] = 0.0
    W[5, 101] = 2.5                     # likewise, alone in its row
    W[9] = 0.0
    W[20, 40:44] = 1e-41
    _check(G, A, W, tile)
    for scale in (2.0 ** 100, 2.0 ** -90):
        _check(G, A, W * np.float32(scale), tile)


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("ea,ew,eg", [(116, -60, 0), (-60, 116, 0), (0, -60, 116), (120, -110, 0), (110, -110, 100)])
def test_large_against_small(ea, ew, eg, tile):
    """Either operand near the top of the fp32 range against one near the bottom: the products are of ordinary size."""
    rng = np.random.default_rng(ea + 2 * ew + 4 * eg + 2000 + tile)
    d_in, d_out = 260, 190
    G, A = _sym(rng, d_out) * np.float32(2.0 ** eg), _sym(rng, d_in) * np.float32(2.0 ** ea)
    err = _check(G, A, (rng.standard_normal((d_out, d_in)) * 2.0 ** ew).astype(np.float32), tile)
    assert err < 1e-6


@pytest.mark.parametrize("tile", [64, 128])
def test_badly_scaled_variables(tile):
    """An inverse whose variables differ by up to 2^15 in scale, with gradients of the inverse scales: all terms of a sum are of
    one size although its factors are not."""
    rng = np.random.default_rng(7 + tile)
    d_in, d_out = 300, 70
    s = np.exp2(rng.integers(-15, 16, d_in)).astype(np.float32)
    A = _sym(rng, d_in) + 4 * np.eye(d_in, dtype=np.float32)
    A = np.ascontiguousarray(A * s[:, None] * s[None, :])
    W = np.ascontiguousarray(rng.standard_normal((d_out, d_in)).astype(np.float32) / s[None, :])
    _check(np.eye(d_out, dtype=np.float32), A, W, tile)


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("place", [0, 37])
@pytest.mark.parametrize("outlier", [2.0 ** 6, 2.0 ** 14, 2.0 ** 20, 2.0 ** 30, 2.0 ** 60])
def test_outliers_keep_the_rest_of_their_row(outlier, place, tile):
    """One element far above the rest of its row, where the row is sampled (0) and where it is not (37 of 391): with identity
    matrices every result is an element of W, rounded to 2^-23 at most.  What is far enough below its row's largest is formed
    again from the operand, so it comes out as it is."""
    rng = np.random.default_rng(place + tile)
    d_in, d_out = 391, 200
    W = rng.standard_normal((d_out, d_in)).astype(np.float32)
    W[::3, place] = outlier
    got = _precondition(np.eye(d_out, dtype=np.float32), np.eye(d_in, dtype=np.float32), W, tile)
    # two roundings of 2^-23, one in each product
    assert np.all(np.abs(got - W) <= 2.0 ** -22 * np.abs(W))


@pytest.mark.parametrize("tile", [64, 128])
def test_ordinary_rows_take_the_two_planes(tile):
    """With identity matrices a result differs from W where h + l does, one value of four; the three planes are exact, and take the
    variables of too different scale, here in powers of two.  (The second contraction, of 32 terms, takes them in any case.)"""
    rng = np.random.default_rng(tile)
    d_in, d_out = 391, 32
    W = rng.standard_normal((d_out, d_in)).astype(np.float32)
    eye = np.eye(d_out, dtype=np.float32)
    assert 0.2 < np.mean(_precondition(eye, np.eye(d_in, dtype=np.float32), W, tile) != W) < 0.3
    s = np.exp2(np.arange(d_in) % 41 - 20).astype(np.float32)
    assert np.array_equal(_precondition(eye, np.diag(s), W / s, tile), W)


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("spread", [8, 10, 12, 20])
def test_spread_of_an_inverse_around_the_limit(spread, tile):
    """Variables of scales 2^0 and 2^spread (squares on the diagonal: the limit lies at 2^11), gradients of the inverse scales."""
    rng = np.random.default_rng(spread + tile)
    d_in, d_out = 300, 70
    s = np.exp2(spread * (np.arange(d_in) % 2)).astype(np.float32)
    A = (_sym(rng, d_in) + 4 * np.eye(d_in, dtype=np.float32)) * s[:, None] * s[None, :]
    W = (rng.standard_normal((d_out, d_in)) / s[None, :]).astype(np.float32)
    got = _precondition(np.eye(d_out, dtype=np.float32), np.ascontiguousarray(A), np.ascontiguousarray(W), tile)
    terms = np.abs(W.astype(np.float64)) @ np.abs(A.astype(np.float64)).T
    err = np.abs(got - W.astype(np.float64) @ A.astype(np.float64).T) / terms
    # roundings of random sign: sqrt(300) 2^-24 of the sum of magnitudes, the largest of 21000 at 5 times that
    assert err.max() <= 5 * np.sqrt(d_in) * 2.0 ** -24


@pytest.mark.parametrize("tile", [64, 128])
def test_gram_rows_of_disjoint_support(tile):
    """Channels that are never active together, channels whose large values meet zeros of the others, channels with one image far
    above the rest and dead ones: every element of the factor to the bound of an fp32 sum of its own terms."""
    N, C, hw = 48, 140, 8
    rng = np.random.default_rng(tile)
    x = rng.standard_normal((N, C, hw, hw)).astype(np.float32)
    x[: N // 2, 0:20] = 0.0
    x[N // 2:, 20:40] = 0.0
    x[:, 40:44] = 0.0
    x[0, 44:50] = 0.0
    x[0, 50:56] *= np.float32(2.0 ** 24)
    x[0, 50:53, 3, 5] = 2.0 ** 30
    x[17, 60:70] *= np.float32(2.0 ** 9)
    L = wl.Layer(N, C, 8, 1, 1, 0, hw, hw, 1)
    with kfac.default_options(force_tile=tile):
        ctx = kfac.Context([L])
    A = torch.empty(C + 1, C + 1, device="cuda")
    kfac.kfac_stats(ctx, [L], kfac.KFAC_F32, [torch.from_numpy(x).cuda()], None, 0.0, True, [A], [torch.empty(8, 8, device="cuda")])
    torch.cuda.synchronize()
    ctx.close()
    m = np.concatenate([x.astype(np.float64).transpose(1, 0, 2, 3).reshape(C, -1), np.ones((1, N * hw * hw))])
    terms = np.abs(m) @ np.abs(m).T / m.shape[1]
    err = np.abs(A.cpu().numpy() - m @ m.T / m.shape[1])
    # roundings of random sign, as above (3072 terms)
    assert np.all(err <= 5 * np.sqrt(m.shape[1]) * 2.0 ** -24 * terms)


@pytest.mark.parametrize("tile", [64, 128])
@pytest.mark.parametrize("hw", [4, 6, 7, 8])
def test_statistics_of_channels_of_different_scale(hw, tile):
    """Factors of a pointwise layer: short runs (the tail path of the main loop), channels from 2^-40 to 2^40, a channel of
    zeros and one with a single element; bias border."""
    N, C = 37, 130
    rng = np.random.default_rng(hw)
    x = rng.standard_normal((N, C, hw, hw)).astype(np.float32) * np.exp2(rng.integers(-40, 41, (1, C, 1, 1))).astype(np.float32)
    x[:, 11] = 0.0
    x[:, 12] = 0.0
    x[20, 12, 1, 2] = 1.5
    L = wl.Layer(N, C, 8, 1, 1, 0, hw, hw, 1)
    with kfac.default_options(force_tile=tile):
        ctx = kfac.Context([L])
    A = torch.empty(C + 1, C + 1, device="cuda")
    kfac.kfac_stats(ctx, [L], kfac.KFAC_F32, [torch.from_numpy(x).cuda()], None, 0.0, True, [A], [torch.empty(8, 8, device="cuda")])
    torch.cuda.synchronize()
    ctx.close()
    m = np.concatenate([x.astype(np.float64).transpose(1, 0, 2, 3).reshape(C, -1), np.ones((1, N * hw * hw))])
    ref = m @ m.T / m.shape[1]
    bound = 5 * np.sqrt(m.shape[1]) * 2.0 ** -24 * (np.abs(m) @ np.abs(m).T) / m.shape[1]   # as in _check
    assert np.all(np.abs(A.cpu().numpy() - ref) <= bound)


def test_time_hardly_depends_on_the_values():
    """512 channels at 7 x 7, 128 samples: images of different size (scales exp(2 N(0,1))), fifth powers of normal values and 5 % of
    dead channels within 1.4 times the time of normal values (measured: 1.0, 1.05 and 1.15; 2.3, 2.3 and 1.6 with scales from four
    places of a row and every tile that holds a row of zeros read twice)."""
    L = wl.conv_layer(128, 512, 512, 3, 1, 1, 7)
    gen = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    act, grad = rnd(128, 512, 7, 7).clamp_(min=0), rnd(128, 512, 7, 7)
    image = torch.exp(2 * rnd(128, 1, 1, 1))
    alive = (torch.rand(1, 512, 1, 1, device="cuda", generator=gen) >= 0.05).float()
    ctx = kfac.Context([L])
    A, G = torch.empty(L.dA, L.dA, device="cuda"), torch.empty(L.dG, L.dG, device="cuda")

    def us(a, g):
        a, g, best = a.contiguous(), g.contiguous(), []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(10):
                kfac.kfac_stats(ctx, [L], kfac.KFAC_F32, [a], [g], 0.0, True, [A], [G])
            e1.record()
            torch.cuda.synchronize()
            best.append(e0.elapsed_time(e1) * 100)
        return min(best)

    normal = us(act, grad)
    times = {"images": us(act * image, grad * image), "powers": us(act ** 5, grad ** 5), "dead": us(act * alive, grad * alive)}
    ctx.close()
    assert max(times.values()) < 1.4 * normal, (normal, times)
