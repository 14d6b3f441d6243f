"""GPU parity for depthwise kernels held four elements a lane: kernel sizes at the edges of a lane's four and of the
teams of 4, 8 and 16 lanes, channel counts at the edges of a workgroup's share, every weight type and output, buffers
that start anywhere, guard bytes around the outputs, alone and in a mixed launch."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


@pytest.fixture(scope="module")
def sq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_07471_amd as sq
    sq.binding.lib()
    return sq


def expect(w, wtype, bits, mode):
    host = w.cpu().numpy() if wtype == "f32" else oracle.widen(w.cpu().view(torch.int16).numpy().view(np.uint16), wtype)
    return oracle.quantize(host, bits, mode)


def outputs(sq, codes, scales):
    deq = codes.astype(np.float32) * scales.reshape(-1, 1, 1, 1)
    return {sq.OUT_INT8: codes, sq.OUT_INT4: oracle.pack_int4(codes), sq.OUT_F32: deq,
            sq.OUT_BF16: torch.from_numpy(deq).to(torch.bfloat16).view(torch.int16).numpy()}


def bits_of(t):
    t = t.cpu()
    return t.view(torch.int16).numpy() if t.dtype == torch.bfloat16 else t.numpy()


# elements 2 ... 64, channels below, at and above the 16, 8 and 4 of a wave
@pytest.mark.parametrize("kh,kw", [(1, 2), (1, 3), (2, 2), (1, 5), (3, 5), (4, 4), (1, 17), (5, 5), (1, 31), (4, 8), (3, 11), (1, 47),
                                   (7, 7), (3, 21), (8, 8)])
@pytest.mark.parametrize("wtype", ["f32", "f16", "bf16"])
def test_alone(sq, kh, kw, wtype):
    gen = torch.Generator().manual_seed(64 * kh + kw)
    for i, cout in enumerate((1, 3, 4, 5, 8, 9, 16, 33, 257)):
        w = torch.randn((cout, 1, kh, kw), generator=gen)
        if i % 3 == 1:
            w = torch.round(w * 2) / 4   # few levels: equal keys, sums of exactly 0 and of exact halves
        if i % 3 == 2:
            w = w * torch.logspace(-32, 32, cout).reshape(-1, 1, 1, 1) if wtype != "f16" else w.abs()
            w[0] = 0
        w = w.to(WTYPES[wtype])
        L = kh * kw
        room = torch.empty(cout * L + 3, dtype=w.dtype, device="cuda")
        d = room[i % 3:i % 3 + cout * L].view(w.shape)   # 16-bit weights at odd half-words too
        d.copy_(w)
        for mode in (sq.MODE_E, sq.MODE_EKC, sq.MODE_EC):
            want = outputs(sq, *expect(w, wtype, 4, mode))
            for out_format, right in want.items():
                flat = torch.from_numpy(np.ascontiguousarray(right)).reshape(-1)
                flat = flat.view(torch.bfloat16) if out_format == sq.OUT_BF16 else flat
                guard = torch.full((flat.numel() + 16,), 77, dtype=flat.dtype, device="cuda")
                out = guard[5:5 + flat.numel()].view(right.shape)
                _, s = sq.squant_quantize_ex(d, 4, mode, out_format, out=out)
                what = (kh, kw, cout, wtype, mode, out_format)
                assert np.array_equal(bits_of(out), right), what
                assert bool((guard[:5] == 77).all()) and bool((guard[5 + flat.numel():] == 77).all()), what


@pytest.mark.parametrize("wtype", ["f32", "bf16"])
def test_in_a_mixed_launch(sq, wtype):
    gen = torch.Generator().manual_seed(5)
    shapes = [(37, 1, 5, 5), (40, 24, 3, 3), (9, 1, 7, 7), (130, 1, 5, 5), (21, 96, 1, 1), (65, 1, 1, 3), (10, 300, 3, 3), (33, 1, 8, 8)]
    for take in (shapes, [s for s in shapes if s[1] != 300]):   # workgroups of two waves and of one
        ws = [torch.randn(s, generator=gen).to(WTYPES[wtype]).cuda() for s in take]
        for mode in (sq.MODE_EK, sq.MODE_EKC):
            codes, scales = sq.BatchPlan(ws).run(4, mode)
            for w, c, s in zip(ws, codes, scales):
                want, want_s = expect(w, wtype, 4, mode)
                assert np.array_equal(c.cpu().numpy(), want) and np.array_equal(s.cpu().numpy(), want_s), (tuple(w.shape), mode)
