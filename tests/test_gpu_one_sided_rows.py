"""GPU parity where many elements of one lane flip: one-sided, constant and few-level values in the
kernels that give a channel to a few lanes (1x1 / FC rows of up to 256 elements, 3x3 channels of up to
32 kernels, depthwise kernels), alone and as members of a mixed launch.  SQuant-C on such a channel
takes more flips than a lane holds elements, so lanes run out of elements before the channel is done."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KINDS = ("constant", "lane_first", "half_normal", "one_sided_grid", "levels")


@pytest.fixture(scope="module")
def sq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_07471_amd as sq
    sq.binding.lib()
    return sq


def values(kind, shape, bits, rng):
    qmax = 2 ** (bits - 1) - 1
    m, row = shape[0], int(np.prod(shape[1:]))
    if kind == "constant":          # as many flips as one-sided quotients of 0.6 ask for, all equal
        w = np.full((m, row), 0.6)
        w[:, -1] = qmax
    elif kind == "lane_first":      # the first lanes' elements rank above all others
        w = np.full((m, row), 0.40)
        for first in range(0, row, 64):   # four elements of each of the first four lanes, vector by vector
            some = w[:, first:first + 16]
            some[:] = 0.49 - 0.005 * rng.integers(0, 2, some.shape)
        w[:, -1] = qmax
    elif kind == "half_normal":
        w = np.abs(rng.standard_normal((m, row)))
    elif kind == "one_sided_grid":
        w = rng.integers(0, 4 * qmax + 1, (m, row)) / 4.0
        w[:, 0] = qmax
    else:                           # "levels": a few distinct weights
        w = rng.choice(np.array([-0.3, 0.2, 0.45, 1.4]), (m, row))
        w[:, 0] = max(qmax, 1.4)
    w[1::2] *= -1
    return w.reshape(shape).astype(np.float32)


def check(sq, shape, other):
    rng = np.random.default_rng(shape[1] * 100 + shape[2])
    for bits in (2, 3, 4, 8):
        for dtype, name in ((torch.float32, None), (torch.float16, "f16")):
            ws = [torch.from_numpy(values(kind, shape, bits, rng)).to(dtype).cuda() for kind in KINDS]
            filler = torch.from_numpy(values("half_normal", other, bits, rng)).to(dtype).cuda()
            for mode in (sq.MODE_EKC, sq.MODE_EC):
                alone = [sq.squant_quantize_ex(w, bits, mode) for w in ws]
                together, scales = sq.squant_quantize_batched_ex([*ws, filler], bits, mode)
                for kind, w, (codes, s), batched, batched_s in zip(KINDS, ws, alone, together, scales):
                    ref = w.cpu().numpy() if name is None else oracle.widen(
                        w.cpu().view(torch.int16).numpy().view(np.uint16), name)
                    want, want_s = oracle.quantize(ref, bits, mode, threads=4)
                    what = (kind, shape, bits, dtype, mode)
                    assert np.array_equal(s.cpu().numpy(), want_s) and np.array_equal(batched_s.cpu().numpy(), want_s), what
                    assert np.array_equal(codes.cpu().numpy(), want), what
                    assert np.array_equal(batched.cpu().numpy(), want), ("mixed", *what)


# rows enough that an odd length is no small tensor; a 3x3 layer makes the batched call a mixed launch
@pytest.mark.parametrize("cin", [4, 10, 13, 16, 31, 32, 48, 63, 64, 100, 128, 130, 200, 255, 256])
def test_short_rows(sq, cin):
    check(sq, (max(40, -(-16384 // cin)), cin, 1, 1), (40, 64, 3, 3))


@pytest.mark.parametrize("cin", [2, 3, 4, 7, 8, 16, 17, 31, 32])
def test_narrow_3x3(sq, cin):
    check(sq, (max(40, -(-16384 // (9 * cin))), cin, 3, 3), (40, 64, 1, 1))


@pytest.mark.parametrize("kh,kw", [(2, 2), (4, 4), (5, 5), (7, 7), (8, 8)])
def test_depthwise(sq, kh, kw):
    check(sq, (67, 1, kh, kw), (40, 64, 3, 3))
