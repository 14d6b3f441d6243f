"""GPU parity for kernels whose perturbations add up to zero exactly: the candidate is the largest |p| of either
sign, the lowest index first.  16-bit weights meet such kernels often.  Every kernel size the register routines are
built for, at channel counts that select each number of kernels per thread, with and without idle lanes, aligned and
not, alone and in a batch."""
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


def zero_sum_weights(shape, rng):
    """Half of the kernels add up to zero: in turn with the largest perturbation negative, positive, and of both
    signs at either order; the others are on a grid of eighths.  The scale is 1 at 4 bits."""
    cout, cin, kh, kw = shape
    K = kh * kw
    w = rng.integers(-48, 49, (cout, cin, K)) / 8.0
    patterns = [[0.375, -0.125, -0.25], [-0.375, 0.125, 0.25], [0.25, -0.25], [-0.25, 0.25]]
    for n in range(0, cin, 2):
        for m in range(cout):
            p = np.zeros(K)
            t = patterns[(n // 2 + m) % 4][:K]
            if abs(sum(t)) < 1e-9:
                p[rng.permutation(K)[:len(t)]] = t
            w[m, n] = p + (rng.integers(-3, 4, K) if m % 3 else 0)
    w[:, -1, 0] = 7.0
    return w.reshape(shape).astype(np.float32)


# (kh, kw): {kernels a thread: channel counts}, for families 9 (3x3) and 5
COUNTS = {
    (3, 3): {1: (3, 20, 33, 63, 64, 129, 130), 2: (66, 96, 128, 257, 300, 363), 4: (192, 200, 248, 255, 256, 392, 512, 513, 1001, 1100, 2050)},
    (1, 2): {1: (3, 33, 64, 129), 2: (65, 128, 300), 4: (200, 255, 500), 8: (363, 512, 2050)},
    (3, 1): {1: (3, 33, 64, 129), 2: (65, 128, 300), 4: (200, 255, 500), 8: (363, 512, 2050)},
    (2, 2): {1: (3, 33, 64, 129), 2: (70, 128, 300), 4: (200, 256, 500), 8: (363, 512, 2050)},
    (1, 5): {1: (3, 33, 64, 129), 2: (65, 128, 300), 4: (200, 256, 513, 1100)},
    (7, 1): {1: (3, 33, 64, 129), 2: (65, 128, 300), 4: (200, 256, 513, 1100)},
    (4, 4): {1: (5, 40, 64, 129, 300)},
    (5, 5): {1: (5, 40, 64, 129, 300)},
    (7, 7): {1: (5, 40, 64, 129, 300)},
}
SHAPES = [(routes.enough(n, kh * kw, 3), n, kh, kw) for (kh, kw), by_kpt in COUNTS.items() for ns in by_kpt.values() for n in ns]
SHAPES += [(6, 3, 4, 4), (6, 3, 7, 7)]   # stems


def test_the_shapes_reach_each_routine():
    want = [(9 if kh == kw == 3 else 5, kpt) for (kh, kw), by_kpt in COUNTS.items() for kpt, ns in by_kpt.items() for _ in ns]
    assert [r[:2] for r in routes.routes(SHAPES)] == want + [(routes.STEM, 0)] * 2


@pytest.mark.parametrize("dtype", ["float32", "float16", "bfloat16"])
def test_zero_sum_kernels(sq, dtype):
    rng = np.random.default_rng(17)
    host = [zero_sum_weights(s, rng) for s in SHAPES]   # eighths below 8: exact in every type
    dev = [torch.from_numpy(w).to(getattr(torch, dtype)).cuda() for w in host]
    for mode in (sq.MODE_EKC, sq.MODE_EC):
        want = [oracle.quantize(w, 4, mode) for w in host]
        batch = sq.BatchPlan(dev).run(4, mode)
        for i, (w, (codes, scales)) in enumerate(zip(dev, want)):
            got = sq.squant_quantize_ex(w, 4, mode)
            for what, (c, s) in (("alone", got), ("batch", (batch[0][i], batch[1][i]))):
                assert np.array_equal(s.cpu().numpy(), scales), (what, w.shape, mode)
                assert np.array_equal(c.cpu().numpy(), codes), (what, w.shape, mode)


@pytest.mark.parametrize("dtype", ["float32", "float16"])
def test_zero_sum_kernels_off_their_alignment(sq, dtype):
    """The same where weights begin one element behind an aligned address, which takes other kernels to any count."""
    rng = np.random.default_rng(18)
    for shape in [s for s in SHAPES if s[1] % 4 == 0]:
        w = zero_sum_weights(shape, rng)
        whole = torch.empty(w.size + 1, dtype=getattr(torch, dtype), device="cuda")
        dev = whole[1:].view(shape)
        dev.copy_(torch.from_numpy(w))
        for mode in (sq.MODE_EKC, sq.MODE_EC):
            codes, scales = oracle.quantize(w, 4, mode)
            c, s = sq.squant_quantize_ex(dev, 4, mode)
            assert np.array_equal(s.cpu().numpy(), scales) and np.array_equal(c.cpu().numpy(), codes), (shape, mode)
