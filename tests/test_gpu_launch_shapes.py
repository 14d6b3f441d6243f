"""GPU parity for 1x1 / FC rows in the launch shapes that few and many rows take: launches that reach each number of
vectors a thread, with and without a tail, in both widths and every output, alone and two lengths in one launch."""
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


VECTORS = (4, 5, 6, 7, 8, 10, 12, 14, 16)
LENGTHS = [4 * v for v in (520, 640, 1000, 1024, 1250, 1536, 1792, 2048, 2560, 3072, 3500, 4096, 6144, 7168, 8192, 9216, 10240, 12288, 14336, 16384)]


def launches(dtype, tail, out_bits):
    """For each number of vectors a thread: a length and a number of rows that get it."""
    whole, bits = (4, 32) if dtype == torch.float32 else (8, 16)
    offs = (0,) if not tail else (-1, -3) if whole == 4 else (-1, -4, -6)   # -4: half a vector of 16-bit weights is left
    sizes = [(n // 8 * 8 + off, rows) for n in LENGTHS for off in offs
             for rows in sorted({8, 300, 2_000_000 // n, 6_000_000 // n, 16_000_000 // n})]
    found = {}
    for size, (nv, _) in zip(sizes, routes.row_shapes([(n, rows, n * rows * (bits + out_bits) // 8, out_bits == 32) for n, rows in sizes])):
        found.setdefault(nv, size)
    assert set(found) == set(VECTORS)
    return found


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("tail", [False, True])
@pytest.mark.parametrize("output", ["int8", "int4", "f32", "bf16"])
def test_each_number_of_vectors(sq, dtype, tail, output):
    gen = torch.Generator().manual_seed(7)
    bits = 6 if output == "int8" else 4
    for nv, (cin, rows) in launches(dtype, tail, {"int8": 8, "int4": 4, "f32": 32, "bf16": 16}[output]).items():
        w = torch.randn((rows, cin, 1, 1), generator=gen).to(dtype)
        out, scales = sq.squant_quantize_ex(w.cuda(), bits, sq.MODE_EKC, sq.OUTPUTS[output])
        codes, want_s = oracle.quantize(host(w), bits, sq.MODE_EKC, threads=8)
        if output == "bf16":
            out, want = out.view(torch.int16), oracle.dequantize_bf16(codes, want_s).view(np.int16)
        else:
            want = {"int8": lambda: codes, "int4": lambda: oracle.pack_int4(codes), "f32": lambda: oracle.dequantize(codes, want_s)}[output]()
        assert np.array_equal(scales.cpu().numpy(), want_s) and np.array_equal(out.cpu().numpy(), want), (nv, cin, rows, output)


def test_two_lengths_in_one_launch(sq):
    gen = torch.Generator().manual_seed(3)
    for shapes in (((7, 16384), (5, 16380), (900, 13005)), ((300, 8192), (3, 7001)), ((6, 36412), (4, 36500))):
        ws = [torch.randn((m, n, 1, 1), generator=gen).cuda() for m, n in shapes]
        codes, scales = sq.BatchPlan(ws).run(3, sq.MODE_EC)
        for w, c, s in zip(ws, codes, scales):
            want, want_s = oracle.quantize(w.cpu().numpy(), 3, sq.MODE_EKC, threads=8)
            assert np.array_equal(c.cpu().numpy(), want) and np.array_equal(s.cpu().numpy(), want_s), tuple(w.shape)
