"""GPU parity for kernels of 10 to 64 elements: two to four of them a channel (the stem of a network, a wave per
channel) and more (4x4 and 7x7 kernels, one per thread), alone and in a batch with other shapes, at the edges of
the workgroup sizes, with rows and buffers at any alignment, and on values that make a kernel flip many elements,
none, or leave its sum exactly zero."""
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


KINDS = ("normal", "grid", "one_sided", "zero_sums", "constant", "scales")


def values(kind, shape, bits, rng):
    qmax = 2 ** (bits - 1) - 1
    if kind == "normal":
        w = rng.standard_normal(shape)
    elif kind == "grid":            # quarters of a step: ties, exact halves, sums of zero
        w = rng.integers(-4 * qmax, 4 * qmax + 1, shape) / 4.0
    elif kind == "one_sided":       # most elements of a kernel have the same sign of perturbation
        w = rng.integers(-qmax, qmax, shape) + 0.4 - 0.1 * rng.random(shape)
        w[1::2] *= -1
    elif kind == "zero_sums":       # pairs of opposite perturbations, the rest whole
        w = rng.integers(-qmax, qmax + 1, shape).astype(np.float64)
        w[..., 0, 0] = 0.25
        w[..., 0, 1] = -0.25
    elif kind == "constant":
        w = np.full(shape, 0.6)
        w[::3] = 0.0
    else:                           # absolute maxima outside the range of the reciprocal
        w = rng.standard_normal(shape)
        w *= np.resize([1e-42, 2.0 ** -80, 1.0, 2.0 ** 80], shape[0]).reshape(-1, 1, 1, 1)
    w.reshape(shape[0], -1)[1, 0] = max(qmax, 1)
    return w.astype(np.float32)


def at_offset(w, elements):
    """w in device memory, `elements` elements behind an allocation's start."""
    buf = torch.zeros(w.numel() + elements, dtype=w.dtype, device="cuda")
    view = buf[elements:].view(w.shape)
    view.copy_(w)
    return view


def check(sq, w, bits, mode, out, s, output, what):
    ref = w.cpu().numpy() if w.dtype == torch.float32 else oracle.widen(
        w.cpu().contiguous().view(torch.int16).numpy().view(np.uint16), "f16" if w.dtype == torch.float16 else "bf16")
    codes, scales = oracle.quantize(ref, bits, mode, threads=8)
    assert np.array_equal(s.cpu().numpy(), scales), what
    want = torch.from_numpy(codes)
    if output == sq.OUT_INT4:
        want = torch.from_numpy(oracle.pack_int4(codes))
    elif output != sq.OUT_INT8:
        want = torch.from_numpy(codes.astype(np.float32) * scales.reshape(-1, 1, 1, 1))
        want = want if output == sq.OUT_F32 else want.to(torch.bfloat16)
    assert torch.equal(out.cpu().reshape(-1), want.reshape(-1)), what


@pytest.mark.parametrize("shape", [(9, 3, 7, 7), (64, 3, 7, 7), (200, 3, 7, 7), (5, 2, 2, 5), (7, 4, 8, 8), (33, 4, 4, 4),
                                   (300, 3, 5, 5), (5, 3, 3, 11), (6, 4, 1, 63), (6, 2, 4, 16)])
def test_stems(sq, shape):
    rng = np.random.default_rng(shape[0] * shape[2])
    for i, kind in enumerate(KINDS):
        for bits in (2, 4, 8):
            dtype = torch.float32 if kind == "scales" else (torch.float32, torch.float16, torch.bfloat16)[(i + bits) % 3]
            w = at_offset(torch.from_numpy(values(kind, shape, bits, rng)).to(dtype), bits % 3)
            other = torch.from_numpy(rng.standard_normal((8, 40, 3, 3)).astype(np.float32)).to(dtype).cuda()
            for mode in (sq.MODE_E, sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
                for output in (sq.OUT_INT8, sq.OUT_INT4 if bits <= 4 else sq.OUT_F32, sq.OUT_BF16):
                    what = f"{kind} {shape} bits={bits} mode={mode} output={output}"
                    check(sq, w, bits, mode, *sq.squant_quantize_ex(w, bits, mode, output), output, what)
                outs, scales = sq.squant_quantize_batched_ex([w, other, w], bits, mode)
                check(sq, w, bits, mode, outs[2], scales[2], sq.OUT_INT8, what + " in a batch")


# cout such that the tensor is no small one (those keep the generic routine)
@pytest.mark.parametrize("k", [4, 7])
@pytest.mark.parametrize("cin", [5, 6, 63, 64, 65, 128, 255, 256, 257, 513, 1024])
def test_one_kernel_per_thread(sq, k, cin):
    shape = (max(3, 16384 // (cin * k * k) + 1), cin, k, k)
    rng = np.random.default_rng(cin)
    for i, kind in enumerate(KINDS):
        bits = (2, 4, 8, 3)[(cin + i) % 4]
        dtype = torch.float32 if kind == "scales" else (torch.float32, torch.float16, torch.bfloat16)[(cin + i) % 3]
        w = at_offset(torch.from_numpy(values(kind, shape, bits, rng)).to(dtype), cin % 4)
        for mode in (sq.MODE_E, sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
            output = (sq.OUT_INT8, sq.OUT_F32, sq.OUT_BF16, sq.OUT_INT4 if bits <= 4 else sq.OUT_INT8)[(i + mode) % 4]
            what = f"{kind} {shape} bits={bits} {dtype} mode={mode} output={output}"
            check(sq, w, bits, mode, *sq.squant_quantize_ex(w, bits, mode, output), output, what)
    other = torch.from_numpy(rng.standard_normal((8, 40, 3, 3)).astype(np.float32)).to(dtype).cuda()
    outs, scales = sq.squant_quantize_batched_ex([other, w], bits, sq.MODE_EKC)
    check(sq, w, bits, sq.MODE_EKC, outs[1], scales[1], sq.OUT_INT8, what + " in a batch")


# 4x4 kernels of up to two waves join a mixed launch, small tensors among them; wider ones and 7x7 get their own
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("cins", [(5, 8, 63, 64), (65, 100, 127, 128), (129, 256, 16, 300)])
def test_members_of_a_batch(sq, cins, dtype):
    rng = np.random.default_rng(cins[0])
    kinds = KINDS if dtype == torch.float32 else KINDS[:-1]
    for i, kind in enumerate(kinds):
        bits = (2, 3, 4, 8)[(i + cins[0]) % 4]
        shapes = [(5, cins[0], 4, 4), (30, cins[1], 4, 4), (9, 40, 3, 3), (5, 8, 7, 7), (3, cins[2], 4, 4), (40, cins[3], 4, 4)]
        ws = [torch.from_numpy(values(kind, s, bits, rng)).to(dtype).cuda() for s in shapes]
        ws[1] = at_offset(ws[1], 1)
        for mode in (sq.MODE_E, sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
            output = (sq.OUT_INT8, sq.OUT_F32, sq.OUT_BF16, sq.OUT_INT4 if bits <= 4 else sq.OUT_INT8)[(i + mode) % 4]
            outs, scales = sq.squant_quantize_batched_ex(ws, bits, mode, output)
            for w, out, s in zip(ws, outs, scales):
                check(sq, w, bits, mode, out, s, output, f"{kind} {tuple(w.shape)} bits={bits} {dtype} mode={mode} output={output}")


@pytest.mark.parametrize("cout", [1, 3, 4, 61, 65])
@pytest.mark.parametrize("cin, side", [(640, 3), (1000, 3), (700, 1), (4000, 1)])
def test_stem_in_a_launch_of_wide_workgroups(sq, cout, cin, side):
    """Three or four channels of a stem share a workgroup, the last of them with fewer."""
    rng = np.random.default_rng(cout)
    shapes = [(cout, 3, 7, 7), (10, cin, side, side), (40, 48, 3, 3), (cout, 2, 5, 5), (8, 800, 3, 3)]
    for kind, bits in (("normal", 4), ("grid", 8), ("one_sided", 3)):
        ws = [torch.from_numpy(values(kind, (max(s[0], 2), *s[1:]), bits, rng)[:s[0]].copy()).cuda() for s in shapes]
        for mode in (sq.MODE_E, sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
            outs, scales = sq.squant_quantize_batched_ex(ws, bits, mode)
            for w, out, s in zip(ws, outs, scales):
                check(sq, w, bits, mode, out, s, sq.OUT_INT8, f"{kind} {tuple(w.shape)} bits={bits} mode={mode}")
