"""GPU parity for kernels of 2, 3, 4, 5, 7 and 9 elements whose codes go to the write-out as whole dwords of four
lanes: channel counts around whole quads and around each number of kernels a thread, packed rows of odd length, values
that make all of a channel's candidates equal, alone and in a mixed launch."""
import numpy as np
import pytest

import oracle
import routes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_07471_amd as sq
    sq.binding.lib()
    return sq


def weights(shape, kind, gen):
    if kind == "normal":
        return torch.randn(shape, generator=gen)
    if kind == "levels":      # equal keys, sums of exactly 0 and of exact halves
        return torch.round(torch.randn(shape, generator=gen) * 3) / 4
    w = torch.full(shape, 0.3)   # every kernel the same: all candidates of a channel are equal
    w[:, 0] = 7.0 if shape[0] % 2 else -7.0
    return w


def check(sq, w, out, s, mode, output):
    host = w.cpu().numpy() if w.dtype == torch.float32 else oracle.widen(w.cpu().view(torch.int16).numpy().view(np.uint16), "f16")
    codes, want_s = oracle.quantize(host, 4, mode, threads=8)
    want = oracle.pack_int4(codes) if output == sq.OUT_INT4 else codes
    assert np.array_equal(s.cpu().numpy(), want_s) and np.array_equal(out.cpu().numpy(), want), (tuple(w.shape), w.dtype, mode, output)


COUNTS = [2, 3, 5, 6, 7, 31, 62, 63, 65, 66, 127, 129, 130, 131, 135, 152, 200, 254, 257, 260, 300, 511, 513, 600, 1021, 1030, 2047, 4095]


@pytest.mark.parametrize("kh,kw", [(1, 2), (3, 1), (2, 2), (1, 5), (7, 1), (3, 3)])
@pytest.mark.parametrize("kind", ["normal", "levels", "equal"])
def test_alone(sq, kh, kw, kind):
    gen = torch.Generator().manual_seed(kh * 8 + kw)
    # no small tensor: odd counts of those stay with the generic routine
    shapes = [(routes.enough(cin, kh * kw, 3) | (1 if i % 3 == 0 else 0), cin, kh, kw) for i, cin in enumerate(COUNTS)]
    assert {family for family, _, _ in routes.routes(shapes)} == {routes.K9 if kh * kw == 9 else routes.SMALL}
    for i, shape in enumerate(shapes):
        w = weights(shape, kind, gen).to(torch.float32 if i % 2 else torch.float16).cuda()
        for mode in (sq.MODE_E, sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
            output = sq.OUT_INT4 if (i + mode) % 2 else sq.OUT_INT8
            out, s = sq.squant_quantize_ex(w, 4, mode, output)
            check(sq, w, out, s, mode, output)


@pytest.mark.parametrize("output", ["INT8", "INT4", "F32"])
def test_narrow_binary32(sq, output):
    """Fewer than 64 kernels a channel: stores that are not aligned, and dwords from 64 on."""
    gen = torch.Generator().manual_seed(5)
    shapes = [(routes.enough(cin, 9, 65), cin, 3, 3) for cin in (33, 35, 36, 48, 60, 61, 63, 64)]
    assert {(family, kpt) for family, kpt, _ in routes.routes(shapes)} == {(routes.K9, 1)}
    for shape in shapes:
        for kind in ("normal", "equal"):
            w = weights(shape, kind, gen).cuda()
            for mode in (sq.MODE_E, sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
                out, s = sq.squant_quantize_ex(w, 4, mode, getattr(sq, "OUT_" + output))
                if output == "F32":
                    codes, want_s = oracle.quantize(w.cpu().numpy(), 4, mode, threads=8)
                    want = codes.astype(np.float32) * want_s.reshape(-1, 1, 1, 1)
                    assert np.array_equal(out.cpu().numpy(), want.reshape(shape)), (shape, kind, mode)
                else:
                    check(sq, w, out, s, mode, getattr(sq, "OUT_" + output))


def test_most_kernels_a_thread(sq):
    gen = torch.Generator().manual_seed(1)
    for shape in ((3, 8192, 1, 2), (3, 8189, 1, 3), (3, 8190, 2, 2), (3, 4094, 1, 7)):
        for kind in ("normal", "equal"):
            w = weights(shape, kind, gen).cuda()
            out, s = sq.squant_quantize_ex(w, 4, sq.MODE_EKC, sq.OUT_INT4)
            check(sq, w, out, s, sq.MODE_EKC, sq.OUT_INT4)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_in_a_mixed_launch(sq, dtype):
    gen = torch.Generator().manual_seed(2)
    shapes = [(routes.enough(n, k, 20), n, 1, k) for n in (3, 31, 67, 130, 258, 301, 500) for k in (2, 3, 5, 7)]
    shapes += [(routes.enough(n, 9, 20), n, 3, 3) for n in (5, 66, 131, 255, 512)]
    assert [family for family, _, _ in routes.routes(shapes)] == [routes.SMALL] * 28 + [routes.K9] * 5
    for kind in ("normal", "levels"):
        ws = [weights(s, kind, gen).to(dtype).cuda() for s in shapes]
        for mode in (sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
            codes, scales = sq.BatchPlan(ws, sq.OUT_INT4).run(4, mode)
            for w, c, s in zip(ws, codes, scales):
                check(sq, w, c, s, mode, sq.OUT_INT4)


@pytest.mark.parametrize("cin", [400, 512])
def test_a_launch_of_many_channels(sq, cin):
    """From 32768 workgroups on, aligned binary32 channels of four kernels a thread in two waves are stored kernel by
    kernel: in a launch of their own and in a mixed one."""
    most = 32768
    assert routes.routes([(most, cin, 3, 3)]) == [(routes.K9, 4, 128)]
    w = torch.randn((most, cin, 3, 3), generator=torch.Generator(device="cuda").manual_seed(cin), device="cuda")
    out, s = sq.squant_quantize_ex(w, 4, sq.MODE_EKC, sq.OUT_INT8)
    few, few_s = sq.squant_quantize_ex(w[:most - 1], 4, sq.MODE_EKC, sq.OUT_INT8)   # whole dwords
    assert torch.equal(out[:most - 1], few) and torch.equal(s[:most - 1], few_s)
    other = torch.randn((64, 256, 1, 1), device="cuda")
    for mode in (sq.MODE_E, sq.MODE_EK, sq.MODE_EKC, sq.MODE_EC):
        codes, scales = sq.BatchPlan([w, other]).run(4, mode)
        check(sq, other, codes[1], scales[1], mode, sq.OUT_INT8)
        out, s = sq.squant_quantize_ex(w, 4, mode, sq.OUT_INT8)
        assert torch.equal(out, codes[0]) and torch.equal(s, scales[0])
        for rows in (slice(0, 200), slice(most - 200, most)):
            check(sq, w[rows], out[rows], s[rows], mode, sq.OUT_INT8)
