"""GPU parity for the threshold search of the 1x1 / FC kernels: channel lengths at the edges of the
vectors per lane and of the workgroup sizes, and values for which the search takes another way
than its first guess: ties by the thousand, a few levels with gaps between them, nearly empty tails, one-sided sums, quotients that the
clamp moves, a scale whose reciprocal is the hardest to round."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_07471_amd as sq
    sq.binding.lib()
    return sq


def overshooting_absmax(qmax, rng):
    """Absolute maxima whose quotient by their own scale exceeds qmax, so that the clamp acts."""
    a = rng.uniform(0.5, 1.0, 200000).astype(np.float32)
    s = a / np.float32(qmax)
    return a[a / s > np.float32(qmax)]


def values(kind, shape, bits, rng):
    qmax = 2 ** (bits - 1) - 1
    m, n = shape
    if kind == "normal":
        w = rng.standard_normal(shape) * 0.05
    elif kind == "grid":        # quotients on a coarse grid: hundreds of equal perturbations, exact halves
        w = rng.integers(-4 * qmax, 4 * qmax + 1, shape) / 4.0
        w[:, 0] = qmax
    elif kind == "one_sided":   # every perturbation has the channel's sign and most of them are equal
        w = rng.integers(-qmax, qmax, shape) + 0.3 + 0.1 * (rng.random(shape) < 0.01)
        w[:, 0] = qmax
        w[1::2] *= -1
    elif kind == "centre":      # a few large weights, the rest far below half a step
        w = rng.standard_normal(shape) * 1e-3
        w[:, ::97] = rng.standard_normal(w[:, ::97].shape)
    elif kind == "outliers":    # one in a hundred sets the scale, the rest crowds around 0
        w = rng.standard_normal(shape) * np.where(rng.random(shape) < 0.01, 4.0, 1.0)
        w[1] = np.abs(w[1])
        w[2, 5] = 60.0
    elif kind == "grid4":       # requantised: a bell of fifteen levels, none of them a level of this scale
        w = np.round(rng.standard_normal(shape) * 2.3).clip(-7, 7) / 7.0
        w[:, 0] = 0.93
        w[1] = np.abs(w[1])
    elif kind == "ternary":     # three levels and the absmax
        w = rng.integers(-1, 2, shape) * 0.37
        w[:, 0] = 1.0
        w[1] = np.abs(w[1])
        w[2, :n // 2] = 0.2
    else:                       # "clamp": absmax elements of both signs with an overshooting quotient
        w = rng.uniform(-0.5, 0.5, shape)
        top = overshooting_absmax(qmax, rng)
        if len(top):
            w[:, 1] = top[:m]
            w[:, -1] = -top[:m]
    return w.astype(np.float32)


# around one vector more per lane, the wave / workgroup border, one, two, four, eight and more waves,
# and the workgroup of 1024 threads with ten to sixteen vectors each
CINS = [260, 512, 516, 1028, 2044, 2048, 2052, 3072, 4096, 6148, 8192, 16384, 24580, 32768,
        33000, 50176, 57347, 65536]


@pytest.mark.parametrize("cin", CINS)
@pytest.mark.parametrize("bits", [2, 4, 8])
def test_matches_the_reference(sq, cin, bits):
    rng = np.random.default_rng(1000 * bits + cin)
    for kind in ("normal", "grid", "one_sided", "centre", "outliers", "clamp", "grid4", "ternary"):
        w = values(kind, (4, cin), bits, rng)
        for dtype, name in ((torch.float32, None), (torch.float16, "f16"), (torch.bfloat16, "bf16")):
            d = torch.from_numpy(w).to(dtype).cuda()
            ref = w if name is None else oracle.widen(
                d.cpu().view(torch.int16).numpy().view(np.uint16).reshape(4, cin, 1, 1), name)
            codes, scales = sq.squant_quantize_ex(d, bits, sq.MODE_EKC)
            want, want_s = oracle.quantize(ref.reshape(4, cin, 1, 1), bits, sq.MODE_EKC)
            what = f"{kind} cin={cin} bits={bits} {dtype}"
            assert np.array_equal(scales.cpu().numpy(), want_s), what
            assert np.array_equal(codes.cpu().numpy().reshape(want.shape), want), what


@pytest.mark.parametrize("cin", [64, 512, 4096])
def test_scale_just_below_a_power_of_two(sq, cin):
    """Scales with an all-ones significand: the reciprocal lies next to a midpoint."""
    rng = np.random.default_rng(cin)
    w = rng.standard_normal((6, cin)).astype(np.float32)
    w = (np.clip(w, -3, 3) / 3).astype(np.float32)
    one = np.float32(2) - np.float32(2) ** -23          # bits = 2: the scale is the absmax itself
    w[:, 0] = one * np.float32(2) ** np.array([0, 1, -20, 30, -40, 50], dtype=np.float32)
    w[:, 1:] *= w[:, :1]
    d = torch.from_numpy(w).cuda()
    codes, scales = sq.squant_quantize(d, 2)
    want, want_s = oracle.quantize(w.reshape(6, cin, 1, 1), 2, sq.MODE_EKC)
    assert np.array_equal(scales.cpu().numpy(), want_s)
    assert np.array_equal(codes.cpu().numpy().reshape(want.shape), want)


@pytest.mark.parametrize("shape", [(64, 64, 1, 1), (64, 512, 1, 1), (16, 4096, 1, 1), (16, 50176, 1, 1), (64, 8, 3, 3),
                                   (64, 128, 3, 3), (64, 301, 3, 3), (64, 128, 1, 3), (64, 64, 5, 5)])
def test_reciprocal_of_the_largest_significand(sq, shape):
    """With a scale of 2 - 2^-23 (at 2 bits the absmax itself) the quotient of 1.0 lies 2^-25 above a half: the
    correctly rounded reciprocal puts it there, the one a unit below puts it on the half, and the code is 0 for 1."""
    one = np.float32(2) - np.float32(2) ** -23
    w = np.ones(shape, np.float32)
    w[:, ::3] = -1.0
    w.reshape(shape[0], -1)[:, 0] = one
    w *= (np.float32(2) ** np.resize([0, 1, -20, 30, -40, 50], shape[0]).astype(np.float32)).reshape(-1, 1, 1, 1)
    codes, scales = sq.squant_quantize(torch.from_numpy(w).cuda(), 2, sq.MODE_E)
    want, want_s = oracle.quantize(w, 2, sq.MODE_E)
    assert np.array_equal(scales.cpu().numpy(), want_s) and np.all(np.abs(want) == 1)
    assert np.array_equal(codes.cpu().numpy(), want)


@pytest.mark.parametrize("dtype,name", [(torch.float32, None), (torch.bfloat16, "bf16")])
@pytest.mark.parametrize("shape", [(24, 1025, 1, 1), (24, 512, 1, 1), (24, 4096, 1, 1), (24, 40000, 1, 1),
                                   (24, 64, 1, 1), (24, 128, 3, 3), (24, 301, 3, 3), (24, 130, 1, 3)])
def test_subnormal_scales(sq, shape, dtype, name):
    """Absolute maxima from 2^-149 to 2^-126: the scale has a few significant bits or is 0, so quotients far
    beyond qmax appear in many elements and every one of them is clamped."""
    rng = np.random.default_rng(shape[1])
    w = rng.uniform(0.05, 1.0, shape) * rng.choice([-1.0, 1.0], shape)
    w.reshape(24, -1)[:, 0] = 1.0
    lowest = -133 if name else -149   # of bfloat16, of binary32
    steps = np.ldexp(1.0, -149 + np.arange(24)).reshape(24, 1, 1, 1)
    w = np.ldexp(np.maximum(np.round(np.abs(w) * steps * 2.0 ** -lowest), 1.0), lowest) * np.sign(w)  # no zeros
    d = torch.from_numpy(w.astype(np.float32)).to(dtype).cuda()
    ref = d.float().cpu().numpy()
    assert np.all(ref != 0)
    for bits in (2, 4, 8):
        for mode in (sq.MODE_EKC, sq.MODE_E):
            codes, scales = sq.squant_quantize_ex(d, bits, mode)
            want, want_s = oracle.quantize(ref, bits, mode, threads=8)
            what = f"{shape} {dtype} bits={bits} mode={mode}"
            assert np.array_equal(scales.cpu().numpy().view(np.uint32), want_s.view(np.uint32)), what
            bad = np.argwhere(codes.cpu().numpy() != want)
            assert len(bad) == 0, f"{what}: {len(bad)} differ, first at {bad[0].tolist()}"


@pytest.mark.parametrize("shape", [(24, 64, 1, 1), (24, 30, 1, 1), (24, 512, 1, 1), (24, 4096, 1, 1), (2, 40000, 1, 1),
                                   (2, 70000, 1, 1), (24, 8, 3, 3), (24, 3, 3, 3), (24, 128, 3, 3), (24, 301, 3, 3),
                                   (64, 130, 1, 3), (24, 64, 5, 5), (24, 1, 3, 3), (24, 1, 5, 5), (24, 16, 7, 7), (2, 5000, 3, 3)])
def test_zero_weights_of_a_zero_scale(sq, shape):
    """Weights of a few 2^-149 at 4 and 8 bits: the scale rounds to 0, every other weight is clamped to +-qmax, a
    weight of 0 keeps the code 0 (0 / 0 must not reach the clamp), and no perturbation is left to flip anything."""
    rng = np.random.default_rng(shape[1])
    units = rng.integers(-3, 4, shape)
    units[:, 0, 0, 0] = 3
    d = torch.from_numpy((units * 2.0 ** -149).astype(np.float32)).cuda()
    for bits in (4, 8):
        want = np.sign(units) * (2 ** (bits - 1) - 1)
        for mode in (sq.MODE_E, sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
            codes, scales = sq.squant_quantize(d, bits, mode)
            together, _ = sq.squant_quantize_batched([d, torch.ones(40, 64, 3, 3, device="cuda"), torch.ones(40, 16, 1, 1, device="cuda")], bits, mode)
            assert not scales.cpu().numpy().any()
            assert np.array_equal(codes.cpu().numpy().reshape(shape), want), (shape, bits, mode)
            assert np.array_equal(together[0].cpu().numpy().reshape(shape), want), ("batched", shape, bits, mode)


@pytest.mark.parametrize("output", ["int8", "int4", "f32", "bf16"])
@pytest.mark.parametrize("wtype", [torch.float32, torch.float16, torch.bfloat16])
def test_every_output_format(sq, wtype, output):
    """Whole rows in each format, one tensor at a time and as members of a mixed launch; enough
    channels that every store of a row meets the next one's data in flight."""
    rng = np.random.default_rng(7)
    ws = [torch.from_numpy(rng.standard_normal((256, cin)).astype(np.float32) * 0.05).to(wtype).cuda()
          for cin in (288, 516, 768, 1280, 2048, 2056, 4096, 16384)]
    fmt = sq.OUTPUTS[output]
    single = [sq.squant_quantize_ex(w, 4, sq.MODE_EKC, fmt) for w in ws]
    together, scales = sq.squant_quantize_batched_ex(ws, 4, sq.MODE_EKC, fmt)
    for w, (out, s), batched, batched_s in zip(ws, single, together, scales):
        shape = (*w.shape, 1, 1)
        ref = w.cpu().numpy().reshape(shape) if wtype == torch.float32 else oracle.widen(
            w.cpu().view(torch.int16).numpy().view(np.uint16).reshape(shape), "f16" if wtype == torch.float16 else "bf16")
        codes, want_s = oracle.quantize(ref, 4, sq.MODE_EKC, threads=8)
        codes = codes.reshape(w.shape)
        value = torch.from_numpy(codes.astype(np.float32) * want_s[:, None])
        want = {"int8": torch.from_numpy(codes), "int4": torch.from_numpy(oracle.pack_int4(codes.reshape(shape))),
                "f32": value, "bf16": value.to(torch.bfloat16)}[output]
        for got, got_s in ((out, s), (batched, batched_s)):
            assert np.array_equal(got_s.cpu().numpy(), want_s)
            assert torch.equal(got.cpu().reshape(want.shape), want), (tuple(w.shape), output, wtype)


@pytest.mark.parametrize("wtype,cin", [(torch.float32, 512), (torch.float32, 516), (torch.float16, 512), (torch.float16, 520),
                                       (torch.bfloat16, 1032)])
def test_channels_walked_by_one_wave(sq, wtype, cin):
    """More than 65536 channels in one launch, with channel counts that no span divides: a wave walks four
    channels up to 512 elements, beyond them two of 16 bits or one of 32.  Each tensor gives what it gives alone,
    where a wave has one channel, and the reference's codes."""
    torch.manual_seed(cin)
    ws = [torch.randn(m, cin, device="cuda").mul_(0.05).to(wtype) for m in (32771, 32769, 1)]
    together, scales = sq.squant_quantize_batched_ex(ws, 4, sq.MODE_EKC)
    for w, codes, s in zip(ws, together, scales):
        alone, alone_s = sq.squant_quantize_ex(w, 4, sq.MODE_EKC)
        assert torch.equal(alone, codes) and torch.equal(alone_s, s)
        ref = w[-5:].float().cpu().numpy()
        want, want_s = oracle.quantize(ref.reshape(*ref.shape, 1, 1), 4, sq.MODE_EKC)
        assert np.array_equal(s[-5:].cpu().numpy(), want_s)
        assert np.array_equal(codes[-5:].cpu().numpy().reshape(want.shape), want)
