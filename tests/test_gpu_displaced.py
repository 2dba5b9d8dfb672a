"""The 13 displaced products of 3x3 convolutions of up to 64 channels, which share a launch: channel counts around the wavefronts'
32 rows, planes that no step of the contraction divides, last parts of a few positions, several layers in one call, and values that lead
single products, or all of them, to the general kernel.  They do so where the split rule (512 positions to a part, 128 parts to a
product) allows the images of a call 256 parts, and, with more than 32 channels in bf16, where these are long: a small layer stands in
the list as often as that takes."""
import pytest
import torch

from paper_2002_06015_amd import kfac, workloads as wl

pytestmark = pytest.mark.gpu


def _times(L, dtype=kfac.KFAC_F32):
    line = -(-(L.w_in + 2) // 8) * 8                    # of a bf16 plane
    K = L.N * (L.h_in + 2) * line
    long = -(-256 * max(900, 13 * line) // K) if dtype == kfac.KFAC_BF16 and L.c_in > 32 else 0
    return max(-(-256 // min(128, L.N * (L.h_in + 2) * (L.w_in + 2) // 512)), long)


def _padded(L):
    """Lines and columns of an fp32 image's plane, as plan_stats pads it."""
    return min(((L.h_in + a, L.w_in + b) for a in range(2, 6) for b in range(2, 6) if (L.h_in + a) * (L.w_in + b) % 4 == 0), key=lambda s: s[0] * s[1])


def _parts(L, times):
    """Contraction length, length of a part and of the last part of an fp32 layer that stands `times` times in a list, for the last one of
    them (parts that are left over go to the first ones): the rule of take_displaced (kfac_api.hip)."""
    Hp, Wp = _padded(L)
    K = L.N * Hp * Wp
    most, rounds = max(-(-K // 4096), min(128, K // max(512, 4 * Wp + 4))), -(-times * K // (8192 * 256))
    assert times * most >= 256
    parts = min(most, max(2, rounds * 256 // times))
    part = -(-(-(-K // parts)) // 32) * 32
    while 32 < (K - 1) % part + 1 < 3 * Wp + 3:
        part += 32
    return K, part, (K - 1) % part + 1


def _factor(layers, dtype, acts, decay=0.75, nhwc=False, fill=None, opts=None):
    gen = torch.Generator(device="cuda").manual_seed(len(layers))
    A = [torch.randn(L.dA, L.dA, device="cuda", generator=gen) for L in layers]
    A = [(a + a.t()).contiguous() for a in A]
    A0 = [a.double() for a in A]
    G = [torch.empty(L.dG, L.dG, device="cuda") for L in layers]
    ctx = kfac.Context(layers, dtype, opts=opts)
    if fill is not None:
        ctx.workspace.fill_(fill)
    kfac.kfac_profile_enable(ctx, True)
    kfac.kfac_stats(ctx, layers, dtype, acts, None, decay, True, A, G, nhwc=nhwc)
    torch.cuda.synchronize()
    together = sum(e["variant"] == 4 and "gemm" in e["kernel"] for e in kfac.kfac_profile_read(ctx))
    ctx.close()
    return A, A0, together


def _patches(x):
    return torch.nn.functional.unfold(x, 3, padding=1).permute(1, 0, 2).reshape(9 * x.shape[1], -1)


def _check(L, x, A, A0, decay=0.75, terms=4096, rows=None):
    """rows: only these, whose products have at most `terms` terms that are not zero."""
    m = _patches(x.double())
    if L.bias:
        m = torch.cat([m, torch.ones(1, m.shape[1], device="cuda", dtype=torch.float64)])
    ref = decay * A0 + (1 - decay) * (m @ m.t()) / m.shape[1]
    # parts of at most 4096 terms, sums of at most 128 parts, 2^-22 a product, and an image's sums less those of its border lines
    # and plus those of its corners (three times the sum of an image at most), three roundings of the running average
    bound = 3 * (terms + 128 + 4) * 2.0 ** -24 * (1 - decay) * (m.abs() @ m.abs().t()) / m.shape[1] + 2.0 ** -22 * A0.abs()
    rows = slice(None) if rows is None else slice(0, rows)
    assert bool(((A.double() - ref).abs() <= bound)[rows].all())
    assert bool((A == A.t()).all())


# (N, c, h, w): K from two parts up; 5 x 5 planes of 49 (fp32: padded so that 4 divides them)
@pytest.mark.parametrize("shape", [(21, 1, 5, 5), (60, 3, 5, 6), (5, 31, 17, 13), (3, 32, 28, 28), (4, 33, 19, 23), (2, 50, 32, 24),
                                   (3, 63, 30, 31), (2, 64, 56, 56), (1, 64, 33, 35), (27, 64, 14, 14)])
@pytest.mark.parametrize("dtype", [kfac.KFAC_F32, kfac.KFAC_BF16])
@pytest.mark.parametrize("bias", [0, 1])
def test_shapes(shape, dtype, bias):
    N, c, h, w = shape
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, bias)
    gen = torch.Generator(device="cuda").manual_seed(sum(shape))
    x = torch.randn(N, c, h, w, device="cuda", generator=gen).clamp_(min=0)
    if dtype == kfac.KFAC_BF16:
        x = x.bfloat16()
    times = _times(L, dtype)
    A, A0, together = _factor([L] * times, dtype, [x] * times)
    assert together == 1
    _check(L, x, A[0], A0[0])
    _check(L, x, A[-1], A0[-1])


SHAPES = [(21, 1, 5, 5), (5, 31, 17, 13), (3, 32, 28, 28), (4, 33, 19, 23), (2, 64, 56, 56), (1, 64, 33, 35)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", [kfac.KFAC_F32, kfac.KFAC_BF16])
def test_whole_numbers(shape, dtype):
    """Sums that fp32 holds exactly: what is left are the roundings of the factor 1 / (N hw)."""
    N, c, h, w = shape
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 1)
    gen = torch.Generator(device="cuda").manual_seed(sum(shape))
    x = torch.randint(-7, 8, (N, c, h, w), device="cuda", generator=gen).float()
    times = _times(L, dtype)
    A, _, together = _factor([L] * times, dtype, [x if dtype == kfac.KFAC_F32 else x.bfloat16()] * times, decay=0.0)
    assert together == 1
    m = _patches(x.double())
    m = torch.cat([m, torch.ones(1, m.shape[1], device="cuda", dtype=torch.float64)])
    ref = m @ m.t() / m.shape[1]
    for a in (A[0], A[-1]):
        assert bool(((a.double() - ref).abs() <= 2.0 ** -22 * ref.abs()).all())


def test_low_planes():
    """Elements 1 + 2^-13, which the high plane holds as 1: without the low plane of one side the sums are 2^-13 off, of both 2^-12."""
    N, c, h, w, times = 9, 20, 51, 51, 6
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 0)
    part = _parts(L, times)[1]
    x = torch.full((N, c, h, w), 1 + 2.0 ** -13, device="cuda")
    A, _, together = _factor([L] * times, kfac.KFAC_F32, [x] * times, decay=0.0)
    assert together == 1
    m = _patches(x.double())
    ref = m @ m.t() / m.shape[1]
    # a rounding of 2^-24 at each of six instructions of a step, for each part and (image, two lines, corner, factor: ten) at the
    # assembly, whose differences are less than a tenth smaller than the sums
    bound = 1.1 * (6 * -(-part // 32) + 85 // 2 + 10) * 2.0 ** -24
    assert bound < 2.0 ** -16
    for a in A:
        assert float(((a.double() - ref) / ref).abs().max()) <= bound


@pytest.mark.parametrize("kind", ["relu", "signed", "scales"])
@pytest.mark.parametrize("shape,times", [((32, 64, 28, 28), 10), ((16, 20, 40, 44), 5), ((40, 33, 30, 32), 5)])
@pytest.mark.parametrize("dtype", [kfac.KFAC_F32, kfac.KFAC_BF16])
def test_errors_against_those_of_single_products(kind, shape, times, dtype):
    """No less accurate than one by one, which a limit of the split rule other than the default leads to: fp32 0.88, bf16 0.96 of their
    error on average over lists.  Single lists vary, with parts up to a quarter longer and so as much more rounding of the sums: 1.3, and
    1.3 squared of the largest error.  (Without the low plane it would be several hundred times.)"""
    N, c, h, w = shape
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 0)
    gen = torch.Generator(device="cuda").manual_seed(sum(shape))
    x = torch.randn(N, c, h, w, device="cuda", generator=gen)
    if kind != "signed":
        x.clamp_(min=0)
    if kind == "scales":
        x *= torch.exp(torch.randn(N, c, 1, 1, device="cuda", generator=gen))
    if dtype == kfac.KFAC_BF16:
        x = x.bfloat16()
    errors = []
    m = _patches(x.double())
    ref = m @ m.t() / m.shape[1]
    for opts, expected in ((None, 1), (kfac.options(target_workgroups=129), 0)):
        A, _, together = _factor([L] * times, dtype, [x] * times, decay=0.0, opts=opts)
        assert together == expected
        e = (A[0].double() - ref).abs() / ref.diagonal().sqrt()[:, None] / ref.diagonal().sqrt()[None, :]
        errors.append((float(e.square().mean().sqrt()), float(e.max())))
    print(kind, shape, dtype, [a / b for a, b in zip(*errors)])
    assert errors[0][0] <= 1.3 * errors[1][0] and errors[0][1] <= 1.69 * errors[1][1]


def test_what_stays_apart():
    """Contractions of one part, 65 channels, and fewer than 256 parts."""
    for N, c, h, w, times in ((2, 64, 14, 14, 256), (4, 65, 28, 28, 40), (32, 64, 56, 56, 1), (4, 32, 30, 30, 31)):
        L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 1)
        x = torch.randn(N, c, h, w, device="cuda").clamp_(min=0)
        A, A0, together = _factor([L] * times, kfac.KFAC_F32, [x] * times)
        assert together == 0
        _check(L, x, A[-1], A0[-1])
    L = wl.Layer(8, 64, 8, 3, 1, 1, 112, 112, 1)         # bf16: short parts of many channels
    x = torch.randn(8, 64, 112, 112, device="cuda").clamp_(min=0).bfloat16()
    assert _factor([L] * 3, kfac.KFAC_BF16, [x] * 3)[2] == 0
    assert _factor([L] * 4, kfac.KFAC_BF16, [x] * 4)[2] == 1


@pytest.mark.parametrize("dtype", [kfac.KFAC_F32, kfac.KFAC_BF16])
@pytest.mark.parametrize("nhwc", [False, True])
def test_several_layers(dtype, nhwc):
    layers = [wl.Layer(6, 40, 8, 3, 1, 1, 28, 28, 1), wl.Layer(6, 64, 8, 3, 1, 1, 20, 22, 0), wl.Layer(6, 16, 8, 1, 1, 0, 9, 9, 1), wl.Layer(6, 5, 8, 3, 1, 1, 60, 17, 1)]
    layers += 15 * layers            # at most 10 + 5 + 13 parts each time
    xs = [torch.randn(L.N, L.c_in, L.h_in, L.w_in, device="cuda").clamp_(min=0) for L in layers]
    if dtype == kfac.KFAC_BF16:
        xs = [x.bfloat16() for x in xs]
    acts = [x.permute(0, 2, 3, 1).contiguous() if nhwc else x for x in xs]
    A, A0, together = _factor(layers, dtype, acts, nhwc=nhwc)
    assert together == 1
    for l, (L, x) in enumerate(zip(layers, xs)):
        if L.k == 3:
            _check(L, x, A[l], A0[l])


@pytest.mark.parametrize("dtype", [kfac.KFAC_F32, kfac.KFAC_BF16])
def test_long_parts(dtype):
    """Parts of more than 4096 positions, in two chains."""
    L = wl.Layer(100, 2, 8, 3, 1, 1, 60, 60, 1)
    x = torch.randn(L.N, L.c_in, L.h_in, L.w_in, device="cuda").clamp_(min=0)
    if dtype == kfac.KFAC_BF16:
        x = x.bfloat16()
    A, A0, together = _factor([L] * 3, dtype, [x] * 3)
    assert together == 1
    _check(L, x, A[0], A0[0])


@pytest.mark.parametrize("shape,times,last", [((97, 64, 28, 28), 2, 4), ((97, 3, 28, 28), 2, 4), ((27, 33, 51, 51), 2, 12), ((9, 20, 51, 51), 6, 4),
                                              ((27, 40, 40, 40), 4, 12), ((9, 50, 72, 72), 3, 4), ((49, 64, 44, 44), 3, 4), ((12, 17, 59, 61), 3, 32),
                                              ((47, 6, 24, 24), 8, 28), ((9, 7, 47, 47), 6, 196), ((27, 50, 32, 24), 8, 668)])
def test_short_last_parts(shape, times, last):
    """Too few positions to take samples from; and lengths behind those that parts are lengthened to avoid.  Nothing behind the image is
    read: the same bits whatever the workspace held."""
    N, c, h, w = shape
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 1)
    assert _parts(L, times)[2] == last
    gen = torch.Generator(device="cuda").manual_seed(sum(shape))
    x = torch.randn(N, c, h, w, device="cuda", generator=gen).clamp_(min=0)
    bits = []
    for fill in (0, 0x7f, 0xff):            # zeros, 3.4e38, NaN
        A, A0, together = _factor([L] * times, kfac.KFAC_F32, [x] * times, fill=fill)
        assert together == 1
        bits.append(A)
    _check(L, x, bits[0][0], A0[0])
    _check(L, x, bits[0][-1], A0[-1])
    for l in range(times):
        assert torch.equal(bits[1][l], bits[0][l]) and torch.equal(bits[2][l], bits[0][l])


# (values that fp16 loses without a scale of their own, beside others of all sizes; more such rows than single products are spared for)
@pytest.mark.parametrize("value", [2.0 ** -60, 2.0 ** -30, 1e-4, 3e5])
@pytest.mark.parametrize("rows", [1, 10, 40])
@pytest.mark.parametrize("other", [1.0, 2.0 ** -40])
def test_rows_that_begin_behind_a_part(value, rows, other):
    """Channels that are zero all through a part of the contraction and not just behind it: the displaced products of the part
    meet elements that the image itself has in the next one only."""
    N, c, h, w, times = 32, 64, 41, 41, 3
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 1)
    K, part, _ = _parts(L, times)
    Hp, Wp = _padded(L)
    gen = torch.Generator(device="cuda").manual_seed(rows)
    x = other * torch.randn(N, c, h, w, device="cuda", generator=gen).clamp_(min=0)
    x[:, :rows] = 0
    found = 0
    for p in range(1, K // part):
        n, at = divmod(p * part, Hp * Wp)
        y, at = at // Wp - (Hp - h), at % Wp - (Wp - w)      # first position of the part, in the image
        if 1 <= y < h and 0 <= at < w - 6:
            x[n, :rows, y, at:at + 6] = value * (1 + torch.rand(rows, 6, device="cuda", generator=gen))
            found += 1
    assert found > 10
    A, A0, together = _factor([L] * times, kfac.KFAC_F32, [x] * times, decay=0.0)
    assert together == 1
    _check(L, x, A[-1], A0[-1], decay=0.0)
    _check(L, x, A[-1], A0[-1], decay=0.0, terms=6 * found, rows=9 * rows)


@pytest.mark.parametrize("shape,times,expected", [((3, 20, 12, 300), 30, 1), ((4, 64, 30, 1000), 8, 1), ((3, 5, 8, 1100), 40, 0), ((2, 40, 200, 210), 8, 1)])
def test_wide_images(shape, times, expected):
    """The displaced images reach hundreds of positions behind a part: parts at least twice as long, or products of their own."""
    N, c, h, w = shape
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 1)
    gen = torch.Generator(device="cuda").manual_seed(sum(shape))
    x = torch.randn(N, c, h, w, device="cuda", generator=gen).clamp_(min=0)
    x *= torch.exp(4 * torch.randn(N, 1, h, 1, device="cuda", generator=gen))
    A, A0, together = _factor([L] * times, kfac.KFAC_F32, [x] * times)
    assert together == expected
    _check(L, x, A[0], A0[0])


# signed: sums near zero, in doubt; dead: rows of zeros; half: too many of them; sparse: rows that sample as zero and are not; scales:
# images of very different size; steep: a row that leaves the range of fp16; far: rows near the ends of fp32; late: images that are black
# down to their middle, so that parts are zero in all rows, or in their own positions only; thin: one element of twenty, no two planes
# in any part; fifth: rows that a few elements dominate
@pytest.mark.parametrize("kind", ["signed", "dead", "half", "sparse", "scales", "steep", "far", "zero", "late", "thin", "fifth"])
@pytest.mark.parametrize("c", [20, 64])
def test_values(kind, c):
    N, h, w = 9, 24, 26
    gen = torch.Generator(device="cuda").manual_seed(c)
    x = torch.randn(N, c, h, w, device="cuda", generator=gen)
    if kind != "signed":
        x.clamp_(min=0)
    if kind == "dead":
        x[:, 3] = 0
    elif kind == "half":
        x[:, ::2] = 0
    elif kind == "sparse":
        x[:, 1] = 0
        x[N - 1, 1, h - 1, 5] = 2.0
        x[:, 7] *= (torch.rand(N, h, w, device="cuda", generator=gen) < 0.01)
    elif kind == "scales":
        x *= torch.exp(4 * torch.randn(N, 1, 1, 1, device="cuda", generator=gen))
    elif kind == "steep":
        x[4, 2, 11, 13] = 2.0 ** 30
    elif kind == "far":
        x[:, 2] *= 2.0 ** 50
        x[:, 5] *= 2.0 ** -50
    elif kind == "zero":
        x.zero_()
    elif kind == "late":
        x[:, :, :h // 2] = 0
    elif kind == "thin":
        x *= torch.rand(N, c, h, w, device="cuda", generator=gen) < 0.1
    elif kind == "fifth":
        x = x ** 5
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 1)
    A, A0, together = _factor([L] * _times(L), kfac.KFAC_F32, [x] * _times(L))
    assert together == 1
    _check(L, x, A[0], A0[0])


def test_infinities():
    """Where an operand is infinite the products are not finite, the others are what they are without it."""
    N, c, h, w = 9, 24, 24, 26
    x = torch.randn(N, c, h, w, device="cuda").clamp_(min=0)
    L = wl.Layer(N, c, 8, 3, 1, 1, h, w, 1)
    whole, _, _ = _factor([L] * _times(L), kfac.KFAC_F32, [x] * _times(L))
    x[3, 6, 10, 10] = float("inf")
    A, _, together = _factor([L] * _times(L), kfac.KFAC_F32, [x] * _times(L))
    assert together == 1
    rows = torch.zeros(L.dA, dtype=torch.bool, device="cuda")
    rows[6 * 9:7 * 9] = True
    touched = rows[:, None] | rows[None, :]
    assert not bool(torch.isfinite(A[0][touched]).any())
    assert bool(torch.isfinite(A[0][~touched]).all())
    assert bool(((A[0] - whole[0])[~touched].abs() <= 1e-5 * whole[0][~touched].abs() + 1e-6).all())
