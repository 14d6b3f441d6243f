"""GPU parity for 1x1 / FC rows in the launch shapes that few and many rows take: lengths that reach each number of
vectors a thread, odd ones among them, alone and two lengths in one launch."""
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


def host(w):
    return w.cpu().numpy() if w.dtype == torch.float32 else oracle.widen(w.cpu().view(torch.int16).numpy().view(np.uint16), "bf16")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cin", [2052, 2561, 3333, 4099, 6247, 7000, 8192, 11001, 13001, 16384, 19001, 23501, 26001, 30001, 34001, 36412, 50176])
def test_rows(sq, cin, dtype):
    gen = torch.Generator().manual_seed(cin)
    for rows in (5, 4_000_000 // cin, 16_000_000 // cin):
        w = torch.randn((rows, cin, 1, 1), generator=gen).to(dtype)
        codes, scales = sq.squant_quantize_ex(w.cuda(), 4, sq.MODE_EKC, sq.OUT_INT8)
        want, want_s = oracle.quantize(host(w), 4, sq.MODE_EKC, threads=8)
        assert np.array_equal(codes.cpu().numpy(), want) and np.array_equal(scales.cpu().numpy(), want_s), (rows, cin, dtype)


def test_two_lengths_in_one_launch(sq):
    gen = torch.Generator().manual_seed(3)
    for shapes in (((7, 16384), (5, 16380), (900, 13005)), ((300, 8192), (3, 7001)), ((6, 36412), (4, 36500))):
        ws = [torch.randn((m, n, 1, 1), generator=gen).cuda() for m, n in shapes]
        codes, scales = sq.BatchPlan(ws).run(3, sq.MODE_EC)
        for w, c, s in zip(ws, codes, scales):
            want, want_s = oracle.quantize(w.cpu().numpy(), 3, sq.MODE_EKC, threads=8)
            assert np.array_equal(c.cpu().numpy(), want) and np.array_equal(s.cpu().numpy(), want_s), tuple(w.shape)
