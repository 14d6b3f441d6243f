"""GPU parity for the kernel that gives four (two) 1x1 / FC channels of 257 to 512 (1024) elements to a
wave: every count of vectors a lane holds, rows that end inside a vector, channel counts that leave
teams of the last wave without a channel, and values whose search ends in each of its ways, in the large
launches that take the kernel by themselves (test_launch_of_its_own; the other lengths and outputs of
test_large_launch take a wave per channel) and as members of a mixed launch (from MIXED_ROWS channels on; fewer
take a wave each)."""
import numpy as np
import pytest

import oracle
from test_gpu_one_sided_rows import KINDS as ONE_SIDED, values as one_sided_values
from test_gpu_threshold_search import values

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SEARCH = ("normal", "grid", "one_sided", "centre", "outliers", "clamp", "grid4", "ternary")


@pytest.fixture(scope="module")
def sq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_07471_amd as sq
    sq.binding.lib()
    return sq


def rows(kind, cin, bits, rng, m):
    w = one_sided_values(kind, (m, cin, 1, 1), bits, rng) if kind in ONE_SIDED else values(kind, (m, cin), bits, rng)
    return w.reshape(m, cin, 1, 1)


def expected(d, bits, mode, output, sq):
    ref = d.cpu().numpy() if d.dtype == torch.float32 else oracle.widen(
        d.cpu().view(torch.int16).numpy().view(np.uint16), "f16" if d.dtype == torch.float16 else "bf16")
    codes, scales = oracle.quantize(ref, bits, mode, threads=8)
    if output == sq.OUT_INT4:
        return torch.from_numpy(oracle.pack_int4(codes)), scales
    if output == sq.OUT_INT8:
        return torch.from_numpy(codes), scales
    value = torch.from_numpy(codes.astype(np.float32) * scales.reshape(-1, 1, 1, 1))
    return value if output == sq.OUT_F32 else value.to(torch.bfloat16), scales


def same(got, want, what):
    assert np.array_equal(got[1].cpu().numpy(), want[1]), what
    assert torch.equal(got[0].cpu().reshape(-1), want[0].reshape(-1)), what


# one more than a vector count holds, its largest, and between; odd rows
@pytest.mark.parametrize("cin", [257, 260, 320, 321, 384, 388, 447, 448, 449, 511, 512, 513, 516, 640, 772, 777, 1001])
def test_large_launch(sq, cin):
    m = 12290   # two teams of the last wave of four have no channel
    rng = np.random.default_rng(cin)
    bits = (2, 3, 4, 8)[cin % 4]
    kinds = SEARCH + ONE_SIDED
    part = -(-m // len(kinds))
    w = np.concatenate([rows(k, cin, bits, rng, part) for k in kinds])[:m]
    for i, dtype in enumerate((torch.float32, torch.float16, torch.bfloat16)):
        d = torch.from_numpy(w).to(dtype).cuda()
        output = (sq.OUT_INT8, sq.OUT_F32, sq.OUT_BF16, sq.OUT_INT4 if bits <= 4 else sq.OUT_INT8)[(cin + i) % 4]
        for mode in (sq.MODE_EKC, sq.MODE_E):
            got = sq.squant_quantize_ex(d, bits, mode, output)
            same(got, expected(d, bits, mode, output, sq), f"cin={cin} {dtype} mode={mode} output={output}")


@pytest.mark.parametrize("cin", [257, 260, 300, 388, 509, 512, 516, 700, 897, 1022, 1024])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
def test_member_of_a_mixed_launch(sq, cin, dtype):
    rng = np.random.default_rng(cin)
    for bits in (2, 4, 8):
        kinds = SEARCH + ONE_SIDED
        ws = [torch.from_numpy(rows(k, cin, bits, rng, 5)).to(dtype).cuda() for k in kinds]
        other = torch.from_numpy(rng.standard_normal((8, 40, 3, 3)).astype(np.float32)).to(dtype).cuda()
        for mode in (sq.MODE_EKC, sq.MODE_EC):
            outs, scales = sq.squant_quantize_batched_ex([*ws, other], bits, mode)
            for kind, w, out, s in zip([*kinds, "3x3"], [*ws, other], outs, scales):
                same((out, s), expected(w, bits, mode, sq.OUT_INT8, sq), f"{kind} cin={cin} {dtype} bits={bits} mode={mode}")


def test_scales_beyond_the_reciprocal_in_one_team_of_a_wave(sq):
    """The teams of a wave have scales of their own: zero, subnormal and huge ones beside ordinary ones."""
    rng = np.random.default_rng(3)
    for cin in (400, 900):
        w = rng.standard_normal((64, cin, 1, 1)).astype(np.float32)
        factor = np.resize(np.float32([1, 0, 1e-42, 2.0 ** -70, 1, 2.0 ** 70, 1e-45, 1, 3e37]), 64)
        d = torch.from_numpy((w * factor.reshape(-1, 1, 1, 1)).astype(np.float32)).cuda()
        other = torch.from_numpy(rng.standard_normal((8, 40, 3, 3)).astype(np.float32)).cuda()
        for bits in (2, 4, 8):
            outs, scales = sq.squant_quantize_batched_ex([d, other], bits, sq.MODE_EKC)
            same((outs[0], scales[0]), expected(d, bits, sq.MODE_EKC, sq.OUT_INT8, sq), f"cin={cin} bits={bits}")


MIXED_ROWS = 2051   # channels from which on a mixed launch solves several a wave, and three teams of the last one


@pytest.mark.parametrize("cin", [257, 300, 388, 509, 512, 516, 700, 897, 1022, 1024])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
def test_several_a_wave_in_a_mixed_launch(sq, cin, dtype):
    rng = np.random.default_rng(cin + 1)
    other = torch.from_numpy(rng.standard_normal((8, 40, 3, 3)).astype(np.float32)).to(dtype).cuda()
    longer = torch.from_numpy(rng.standard_normal((9, 1500, 1, 1)).astype(np.float32)).to(dtype).cuda()   # a wave each
    for bits in (2, 4, 8):
        kinds = SEARCH + ONE_SIDED
        part = -(-MIXED_ROWS // len(kinds))
        w = np.concatenate([rows(k, cin, bits, rng, part) for k in kinds])[:MIXED_ROWS]
        if dtype == torch.float32:   # scales of their own in the teams of a wave
            factor = np.resize(np.float32([1, 0, 1e-42, 2.0 ** -70, 1, 2.0 ** 70, 1e-45, 1, 1, 1, 1]), len(w))
            w = (w * factor.reshape(-1, 1, 1, 1)).astype(np.float32)
        ws = [other, torch.from_numpy(w).to(dtype).cuda(), longer]
        for mode in (sq.MODE_EKC, sq.MODE_E):
            output = sq.OUT_INT4 if bits <= 4 and mode == sq.MODE_EKC else sq.OUT_INT8
            outs, scales = sq.squant_quantize_batched_ex(ws, bits, mode, output)
            for what, x, out, s in zip(("3x3", "rows", "longer"), ws, outs, scales):
                same((out, s), expected(x, bits, mode, output, sq), f"{what} cin={cin} {dtype} bits={bits} mode={mode}")


# every kernel of a launch of its own that takes several rows a wave, with the fewest channels it is chosen for (and
# two more: teams of the last wave have no channel)
@pytest.mark.parametrize("dtype, mode, cin, m, outputs", [
    ("float32", "EKC", 257, 12290, "int8 int4 f32"), ("float32", "EKC", 320, 16386, "int4 bf16 f32"),
    ("float32", "EC", 381, 16386, "int8 bf16 f32"), ("float32", "EKC", 448, 16386, "int8 bf16"),
    ("float32", "EKC", 449, 16386, "int4"), ("float32", "EC", 512, 16386, "int8"),
    ("float32", "EKC", 513, 12290, "int4"), ("float32", "EC", 640, 24578, "int8 bf16"),
    ("float32", "EKC", 767, 12290, "int8"), ("float32", "EKC", 895, 24578, "int4 bf16"),
    ("float32", "EKC", 1022, 24578, "int8"), ("float32", "E", 320, 16386, "int8 int4 bf16"),
    ("float32", "E", 381, 12290, "int8"),
    ("float16", "EKC", 257, 12290, "int4 f32"), ("bfloat16", "EC", 384, 16386, "int8 bf16"),
    ("float16", "EKC", 509, 16386, "int4 bf16"), ("bfloat16", "EKC", 512, 16386, "int8 bf16"),
    ("bfloat16", "EKC", 771, 24578, "int8 int4"), ("float16", "EC", 1023, 24578, "int4"),
    ("bfloat16", "E", 383, 16386, "int8 bf16"), ("float16", "E", 511, 16386, "int4 bf16"),
    ("float16", "E", 777, 24578, "int8"), ("bfloat16", "E", 1021, 24578, "int4")])
def test_launch_of_its_own(sq, dtype, mode, cin, m, outputs):
    rng = np.random.default_rng(cin + m)
    kinds = SEARCH + ONE_SIDED
    part = -(-m // len(kinds))
    for output in outputs.split():
        bits = {"int4": 4, "int8": 8, "f32": 3, "bf16": 2}[output]
        w = np.concatenate([rows(k, cin, bits, rng, part) for k in kinds])[:m]
        d = torch.from_numpy(w).to(getattr(torch, dtype)).cuda()
        got = sq.squant_quantize_ex(d, bits, sq.MODES[mode], sq.OUTPUTS[output])
        same(got, expected(d, bits, sq.MODES[mode], sq.OUTPUTS[output], sq), f"cin={cin} {dtype} mode={mode} output={output}")


# Scales of 2 * 2^-149 under which every weight is a half step from a code: each perturbation is 2^22 in units of
# 2^-23, all of one sign, so 512 of them sum to 2^31 either way.  absmax / qmax rounds to 2 for each multiple.
@pytest.mark.parametrize("bits, multiples", [(3, (5, 7)), (4, (11, 13)), (5, (23, 27)), (6, (47, 61)), (8, (191, 253))])
@pytest.mark.parametrize("cin", [511, 512, 1024])
def test_every_element_on_a_half_step(sq, bits, multiples, cin):
    lead = np.resize(np.float32([multiples[0], -multiples[0], multiples[1], -multiples[1], 3]), 16386)
    step = np.uint32(1).view(np.float32)   # 2^-149
    d = torch.from_numpy(np.repeat((lead * step)[:, None], cin, axis=1).reshape(-1, cin, 1, 1)).cuda()
    other = torch.from_numpy(np.random.default_rng(cin).standard_normal((8, 40, 3, 3)).astype(np.float32)).cuda()
    for mode in (sq.MODE_EKC, sq.MODE_EC):
        want = expected(d, bits, mode, sq.OUT_INT8, sq)
        same(sq.squant_quantize_ex(d, bits, mode, sq.OUT_INT8), want, f"cin={cin} bits={bits} mode={mode}")
        for m in (83, MIXED_ROWS):
            outs, scales = sq.squant_quantize_batched_ex([d[:m].contiguous(), other], bits, mode)
            same((outs[0], scales[0]), (want[0][:m], want[1][:m]), f"mixed, {m} of cin={cin} bits={bits} mode={mode}")
