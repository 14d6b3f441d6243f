"""GPU parity for channel counts that are no multiple of four and for weights and outputs that start
anywhere: the register kernels that read and write rows through range-checked descriptors.  Channel
counts lie next to the edges of vectors, waves and kernels per thread; buffers start off every
alignment; guard bytes around the outputs must stay as they were."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

OUT_DTYPE = {"int8": torch.int8, "int4": torch.uint8, "f32": torch.float32, "bf16": torch.bfloat16}


@pytest.fixture(scope="module")
def sq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_07471_amd as sq
    sq.binding.lib()
    return sq


def weights(shape, rng, kind):
    if kind == "grid":   # equal perturbations, exact halves, kernels whose sum is zero
        w = rng.integers(-28, 29, shape) / 4.0
        w.reshape(shape[0], -1)[:, 0] = 7.0
    else:
        w = rng.standard_normal(shape) * 0.05
        if shape[0] > 2:
            w[2] = 0.0
    return w.astype(np.float32)


def expected(codes, scales, output):
    value = codes.astype(np.float32) * scales.reshape(-1, 1, 1, 1)
    if output == "int8":
        return torch.from_numpy(codes)
    if output == "int4":
        return torch.from_numpy(oracle.pack_int4(codes))
    return torch.from_numpy(value).to(OUT_DTYPE[output])


def run_off_alignment(sq, w, wtype, bits, mode, output, lead):
    """One tensor whose weights start `lead` elements, and whose output `lead` elements, into their buffers."""
    flat = torch.zeros(w.size + lead + 8, dtype=wtype, device="cuda")
    dw = flat[lead:lead + w.size].view(w.shape)
    dw.copy_(torch.from_numpy(w))
    row = w.size // w.shape[0]
    n = w.shape[0] * ((row + 1) // 2) if output == "int4" else w.size
    guard = torch.full((n + lead + 64,), 77, dtype=OUT_DTYPE[output], device="cuda")
    out = guard[lead:lead + n]
    scales = torch.empty(w.shape[0], dtype=torch.float32, device="cuda")
    sq.squant_quantize_ex(dw, bits, sq.MODES[mode], sq.OUTPUTS[output], out, scales)
    host = guard.cpu()
    assert bool((host[:lead] == 77).all()) and bool((host[lead + n:] == 77).all()), "wrote outside its output"
    if wtype != torch.float32:
        w = oracle.widen(dw.contiguous().cpu().view(torch.int16).numpy().view(np.uint16),
                         "f16" if wtype == torch.float16 else "bf16")
    codes, want_s = oracle.quantize(w, bits, oracle_mode(mode))
    return host[lead:lead + n], scales.cpu().numpy(), codes, want_s


def oracle_mode(mode):
    return {"E": 0, "EK": 1, "EKC": 2, "EC": 3}[mode]


# the small-kernel cases carry enough channels not to count as a small tensor (those stay generic)
CASES = ([(3, 3, n) for n in (2, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 63, 65, 66, 127, 130, 153, 255, 257, 511, 514, 1023, 1025, 4095)] +
         [(1, 1, n) for n in (1, 2, 3, 5, 13, 17, 30, 33, 63, 65, 101, 127, 130, 255, 257, 511, 514, 1023, 2047, 2049, 4095, 6147, 9001, 32766, 57347)] +
         [(1, 3, 2), (3, 1, 85), (1, 7, 33), (7, 1, 129), (2, 2, 63), (2, 2, 514), (1, 5, 67), (5, 5, 3), (5, 5, 65),
          (1, 2, 301), (1, 7, 1023)])


@pytest.mark.parametrize("kh,kw,cin", CASES)
def test_odd_channel_counts(sq, kh, kw, cin):
    rng = np.random.default_rng(cin * 100 + kh * 10 + kw)
    lead = 0
    for wtype in (torch.float32, torch.float16, torch.bfloat16):
        for output, bits, mode in (("int8", 4, "EKC"), ("int4", 4, "EKC"), ("f32", 3, "EK"), ("bf16", 8, "EKC"),
                                   ("int8", 8, "EC"), ("int4", 2, "E")):
            w = weights((max(4, -(-16384 // (cin * kh * kw))) if cin < 400 else 4, cin, kh, kw), rng,
                        "grid" if lead % 2 else "normal")
            lead = (lead + 1) % 8
            got, got_s, codes, want_s = run_off_alignment(sq, w, wtype, bits, mode, output, lead)
            what = (kh, kw, cin, wtype, output, bits, mode, lead)
            assert np.array_equal(got_s, want_s), what
            want = expected(codes, want_s, output).reshape(-1)
            assert torch.equal(got.view(torch.int16) if output == "bf16" else got,
                               want.view(torch.int16) if output == "bf16" else want), what


@pytest.mark.parametrize("wtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("mode", ["E", "EK", "EKC", "EC"])
def test_packed_checkpoint_in_one_call(sq, wtype, mode):
    """Layers of a pruned network, weights in one buffer without padding, as one batched call."""
    rng = np.random.default_rng(5)
    shapes = [(45, 3, 7, 7), (45, 45, 3, 3), (181, 45, 1, 1), (90, 181, 1, 1), (90, 90, 3, 3), (33, 90, 1, 7),
              (363, 1, 3, 3), (17, 33, 5, 5), (363, 909, 1, 1), (100, 363, 3, 3), (50, 1454, 1, 1), (1000, 2909, 1, 1)]
    ws = [weights(s, rng, "normal") for s in shapes]
    flat = torch.from_numpy(np.concatenate([w.reshape(-1) for w in ws])).to(wtype).cuda()
    views, at = [], 0
    for w in ws:
        views.append(flat[at:at + w.size].view(w.shape))
        at += w.size
    outs, scales = sq.squant_quantize_batched_ex(views, 4, sq.MODES[mode], sq.OUT_INT4)
    for v, out, s in zip(views, outs, scales):
        host = v.contiguous().cpu()
        w = host.numpy() if wtype == torch.float32 else oracle.widen(host.view(torch.int16).numpy().view(np.uint16), "bf16")
        codes, want_s = oracle.quantize(w, 4, oracle_mode(mode), threads=4)
        assert np.array_equal(s.cpu().numpy(), want_s), tuple(v.shape)
        assert np.array_equal(out.cpu().numpy(), oracle.pack_int4(codes)), tuple(v.shape)


@pytest.mark.parametrize("kh,kw", [(1, 2), (2, 2), (1, 7), (4, 4), (1, 17), (5, 5), (4, 8), (3, 11), (7, 7), (8, 8), (5, 13)])
def test_depthwise_kernels(sq, kh, kw):
    """One kernel per channel: teams of 16, 32 and 64 lanes at their edges (65 elements: the generic kernel)."""
    rng = np.random.default_rng(kh * 100 + kw)
    for lead, (wtype, output, bits, mode) in enumerate([
            (torch.float32, "int8", 4, "EKC"), (torch.float16, "int4", 4, "EK"), (torch.bfloat16, "f32", 8, "EC"),
            (torch.float32, "bf16", 2, "EC"), (torch.float32, "int4", 3, "EC"), (torch.bfloat16, "int8", 5, "E")]):
        for kind in ("grid", "normal"):
            w = weights((67, 1, kh, kw), rng, kind)
            got, got_s, codes, want_s = run_off_alignment(sq, w, wtype, bits, mode, output, lead)
            what = (kh, kw, wtype, output, bits, mode, kind)
            assert np.array_equal(got_s, want_s), what
            want = expected(codes, want_s, output).reshape(-1)
            assert torch.equal(got.view(torch.int16) if output == "bf16" else got,
                               want.view(torch.int16) if output == "bf16" else want), what
