"""GPU parity for kernels whose perturbations add up to zero exactly: the candidate is the largest |p| of either
sign, the lowest index first.  16-bit weights meet such kernels often.  Every kernel size the register routines are
built for, at channel counts that select each number of kernels per thread, with and without idle lanes, alone and in
a batch."""
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


SHAPES = [(9, 3, 3, 3), (8, 20, 3, 3), (6, 63, 3, 3), (6, 96, 3, 3), (6, 130, 3, 3), (5, 248, 3, 3), (5, 301, 3, 3),
          (4, 512, 3, 3), (3, 1001, 3, 3), (7, 40, 1, 3), (5, 129, 2, 2), (5, 300, 1, 7), (5, 70, 5, 5), (6, 40, 4, 4),
          (5, 9, 7, 7), (6, 3, 7, 7)]


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
