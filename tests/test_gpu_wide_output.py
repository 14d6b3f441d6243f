"""GPU parity for 16-bit rows written as binary32: the lanes of a row exchange their codes, so that each store is
consecutive.  Lengths at the edges of whole vectors of eight and of the launch shapes, for a workgroup, a wave and a
part of a wave to a row, rows that start anywhere."""
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


def check(sq, w, out, s, mode, what):
    codes, scales = oracle.quantize(oracle.widen(w.cpu().view(torch.int16).numpy().view(np.uint16), "bf16"), 4, mode, threads=8)
    assert np.array_equal(s.cpu().numpy(), scales), what
    assert np.array_equal(out.cpu().numpy(), codes.astype(np.float32) * scales.reshape(-1, *[1] * (w.dim() - 1))), what


# a wave a row (257 to 2048), a workgroup of one to sixteen waves, ten and more vectors a thread
@pytest.mark.parametrize("cin", [257, 264, 391, 392, 511, 512, 513, 520, 1016, 1023, 1031, 1032, 2040, 2041, 2049, 2056, 3072,
                                 4089, 4096, 4104, 8193, 8200, 16384, 24583, 33001, 50176, 65536])
def test_rows(sq, cin):
    gen = torch.Generator().manual_seed(cin)
    w = torch.randn((5, cin, 1, 1), generator=gen).to(torch.bfloat16).cuda()
    for mode in (sq.MODE_E, sq.MODE_EKC):
        guard = torch.full((5 * cin + 16,), -7.0, device="cuda")   # nothing is written around the rows
        out = guard[8:8 + 5 * cin].view(w.shape)
        _, s = sq.squant_quantize_ex(w, 4, mode, sq.OUT_F32, out=out)
        check(sq, w, out, s, mode, (cin, mode))
        assert bool((guard[:8] == -7.0).all()) and bool((guard[-8:] == -7.0).all()), (cin, mode)


# several rows a wave: a launch of its own (from 12288 channels on) and members of a mixed launch (from 2048 on)
@pytest.mark.parametrize("cin", [257, 263, 264, 320, 513, 519, 520, 777, 1017, 1024])
def test_rows_that_share_a_wave(sq, cin):
    gen = torch.Generator().manual_seed(cin)
    if cin <= 320:
        w = torch.randn((12290, cin, 1, 1), generator=gen).to(torch.bfloat16).cuda()
        out, s = sq.squant_quantize_ex(w, 4, sq.MODE_EKC, sq.OUT_F32)
        check(sq, w, out, s, sq.MODE_EKC, cin)
    ws = [torch.randn(sh, generator=gen).to(torch.bfloat16).cuda() for sh in ((2051, cin, 1, 1), (6, 24, 3, 3))]
    codes, scales = sq.BatchPlan(ws, sq.OUT_F32).run(4, sq.MODE_EKC)
    for w, c, s in zip(ws, codes, scales):
        check(sq, w, c, s, sq.MODE_EKC, ("batch", cin, tuple(w.shape)))
