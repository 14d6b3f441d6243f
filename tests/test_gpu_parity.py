"""GPU parity: the HIP path against the CPU reference solver, element by element,
bit-exact for int8 codes and for the binary32 scales (compared as bit patterns)."""
import numpy as np
import pytest

import oracle
from paper_2202_07471_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_07471_amd as sq
    sq.binding.lib()          # raises if the HIP library is missing: no fallback
    return sq


def assert_same(codes_gpu, scales_gpu, w, bits, mode, threads=8, what=""):
    want_c, want_s = oracle.quantize(w, bits, mode, threads=threads)
    got_c = codes_gpu.cpu().numpy().reshape(want_c.shape)
    got_s = scales_gpu.cpu().numpy()
    assert np.array_equal(got_s.view(np.uint32), want_s.view(np.uint32)), f"scales differ {what}"
    if not np.array_equal(got_c, want_c):
        bad = np.argwhere(got_c != want_c)
        raise AssertionError(f"codes differ {what}: {len(bad)} elements, first at {bad[0].tolist()} "
                             f"gpu={got_c[tuple(bad[0])]} ref={want_c[tuple(bad[0])]}")


def run_single(sq, w, bits, mode):
    dw = torch.from_numpy(w).cuda()
    codes, scales = sq.squant_quantize(dw, bits, mode)
    torch.cuda.synchronize()
    return codes, scales


def rand_weights(shape, seed, kind="normal"):
    rng = np.random.default_rng(seed)
    if kind == "normal":
        return (rng.standard_normal(shape) * 0.05).astype(np.float32)
    if kind == "heavy":
        return (rng.standard_t(3, shape) * 0.05).astype(np.float32)
    if kind == "grid":      # coarse grid: many equal perturbations, exact halves, zero sums
        w = rng.integers(-28, 29, shape).astype(np.float32) / 4.0
        w.reshape(shape[0], -1)[:, 0] = 7.0
        return w
    raise ValueError(kind)


# ---------------------------------------------------------------------------
# config 1: one [64,64,3,3] tensor, every mode and bit width
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("bits", [2, 3, 4, 5, 6, 8])
def test_config1_all_modes_and_bits(sq, mode, bits):
    w = synth.generate(synth.config_specs(1)[0])
    codes, scales = run_single(sq, w, bits, mode)
    assert_same(codes, scales, w, bits, mode, what=f"C1 bits={bits} mode={mode}")


# ---------------------------------------------------------------------------
# shapes that span several tiles, ragged tails and the degenerate cases
# ---------------------------------------------------------------------------
SHAPES = [
    (1, 1, 1, 1), (1, 1, 3, 3), (3, 1, 3, 3), (96, 1, 3, 3),      # depthwise-like, M = 1
    (5, 3, 7, 7), (64, 3, 7, 7), (7, 2, 5, 5), (4, 5, 11, 11),   # large kernels
    (33, 17, 3, 3), (64, 64, 3, 3), (31, 130, 3, 3), (8, 600, 3, 3), (4, 1100, 3, 3),
    (10, 1, 1, 1), (17, 63, 1, 1), (1000, 512, 1, 1), (12, 2048, 1, 1), (3, 5000, 1, 1),
    (9, 100, 2, 2), (6, 37, 1, 3), (5, 50, 4, 4), (2, 3000, 3, 3),
    (7, 100, 1, 1), (7, 1028, 1, 1), (5, 4096, 1, 1), (3, 8192, 1, 1), (2, 32768, 1, 1),
    (2, 32764, 1, 1), (2, 26000, 1, 1), (3, 20000, 1, 1), (40, 16, 1, 1), (6, 128, 3, 3), (6, 96, 3, 3), (6, 192, 3, 3), (3, 4096, 3, 3),
]


@pytest.mark.parametrize("kind", ["normal", "heavy", "grid"])
@pytest.mark.parametrize("shape", SHAPES)
def test_shapes_ekc(sq, shape, kind):
    w = rand_weights(shape, seed=sum(shape) * 7 + len(kind), kind=kind)
    for mode in (2, 1):
        codes, scales = run_single(sq, w, 4, mode)
        assert_same(codes, scales, w, 4, mode, what=f"{shape} {kind} mode={mode}")


@pytest.mark.parametrize("bits", [3, 8])
@pytest.mark.parametrize("shape", [(33, 17, 3, 3), (17, 63, 1, 1), (5, 3, 7, 7), (96, 1, 3, 3)])
def test_shapes_other_bits(sq, shape, bits):
    for kind in ("normal", "heavy"):
        w = rand_weights(shape, seed=bits + sum(shape), kind=kind)
        for mode in (0, 2, 3):
            codes, scales = run_single(sq, w, bits, mode)
            assert_same(codes, scales, w, bits, mode, what=f"{shape} {kind} bits={bits} mode={mode}")


def test_zero_and_constant_channels(sq):
    w = rand_weights((8, 20, 3, 3), 3)
    w[0] = 0.0                      # all-zero channel: scale 1, codes 0
    w[1] = 0.25                     # constant channel: every x = qmax
    w[2] = -1e-30                   # tiny magnitudes
    w[3, 1:] = 0.0                  # one non-zero kernel
    w[4] = 0.0
    w[4, 3, 1, 1] = -2.0            # a single non-zero element
    for mode in (0, 1, 2, 3):
        codes, scales = run_single(sq, w, 4, mode)
        assert_same(codes, scales, w, 4, mode, what=f"special channels mode={mode}")
    assert float(scales[0]) == 1.0 and int(codes[0].abs().max()) == 0


@pytest.mark.parametrize("shape", [(24, 64, 3, 3), (24, 96, 1, 1), (24, 10, 2, 2)])
def test_extreme_magnitudes(sq, shape):
    """Channels whose absmax sits far outside the usual range (down to subnormal scales, up to
    near overflow, and just either side of the kernels' internal range switch at 2^-60 / 2^60),
    with a sprinkling of elements ~2^-110 times smaller than the rest."""
    rng = np.random.default_rng(99)
    w = rng.standard_normal(shape).astype(np.float64)
    tiny = rng.random(shape) < 0.1
    w[tiny] *= 2.0 ** -110
    exps = [-140, -127, -120, -100, -61, -60, -59, -30, 0, 30, 59, 60, 61, 100, 120, 125,
            -62, -58, 58, 62, -90, 90, -10, 10]
    for m, e in enumerate(exps):
        w[m] = np.ldexp(w[m], e)
    w = np.clip(w, -3e38, 3e38).astype(np.float32)
    for bits in (4, 8):
        for mode in (2, 0):
            codes, scales = run_single(sq, w, bits, mode)
            assert_same(codes, scales, w, bits, mode, what=f"extreme {shape} bits={bits} mode={mode}")


def test_unaligned_views(sq):
    """Channel lengths that leave the output channel base misaligned for wide access."""
    for shape in [(7, 3, 3, 3), (5, 7, 1, 1), (9, 5, 1, 3)]:
        w = rand_weights(shape, 5)
        codes, scales = run_single(sq, w, 4, 2)
        assert_same(codes, scales, w, 4, 2, what=f"unaligned {shape}")


def test_deterministic(sq):
    w = synth.generate(synth.TensorSpec(60, 0, (256, 256, 3, 3), "student_t3", 0.03))
    a = run_single(sq, w, 4, 2)
    b = run_single(sq, w, 4, 2)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


# ---------------------------------------------------------------------------
# layer sets through the batched entry point (configs 2, 3, 4)
# ---------------------------------------------------------------------------
def run_batched(sq, ws, bits, mode):
    dws = [torch.from_numpy(w).cuda() for w in ws]
    plan = sq.BatchPlan(dws)
    codes, scales = plan.run(bits, mode)
    torch.cuda.synchronize()
    return codes, scales


@pytest.mark.parametrize("config,bits", [(2, 4), (3, 4), (3, 8), (4, 4), (6, 4)])
def test_layer_sets_batched(sq, config, bits):
    specs = synth.config_specs(config)
    ws = [synth.generate(s) for s in specs]
    codes, scales = run_batched(sq, ws, bits, 2)
    for s, w, c, sc in zip(specs, ws, codes, scales):
        assert_same(c, sc, w, bits, 2, what=f"config {config} tensor {s.index} {s.shape} bits={bits}")


def test_batched_equals_single_and_other_modes(sq):
    specs = synth.config_specs(4)[:12] + synth.config_specs(2)[:3]
    ws = [synth.generate(s) for s in specs]
    for mode in (0, 1, 3):
        codes, scales = run_batched(sq, ws, 4, mode)
        for s, w, c, sc in zip(specs, ws, codes, scales):
            assert_same(c, sc, w, 4, mode, what=f"batched mode={mode} {s.shape}")
            c1, s1 = run_single(sq, w, 4, mode)
            assert torch.equal(c1, c) and torch.equal(s1, sc)


def test_mixed_launch_with_every_variant_and_large_members(sq):
    """One batched call whose tensors cover every kernel variant: the small ones share one
    mixed launch, the ones that need more than 256 threads per channel keep their own."""
    shapes = [(6, 64, 3, 3), (5, 96, 3, 3), (4, 512, 3, 3), (3, 1024, 3, 3), (2, 2048, 3, 3),
              (9, 128, 1, 1), (7, 512, 1, 1), (5, 2048, 1, 1), (3, 8192, 1, 1), (2, 32768, 1, 1),
              (33, 17, 3, 3), (96, 1, 3, 3), (5, 3, 7, 7), (3, 5000, 1, 1), (4, 6, 11, 11),
              (17, 63, 1, 1), (6, 64, 3, 3), (1, 1, 1, 1)]
    ws = [rand_weights(sh, 400 + i, "heavy" if i % 3 == 0 else "normal") for i, sh in enumerate(shapes)]
    for bits, mode in ((4, 2), (3, 1), (8, 3), (4, 0)):
        codes, scales = run_batched(sq, ws, bits, mode)
        for sh, w, c, sc in zip(shapes, ws, codes, scales):
            assert_same(c, sc, w, bits, mode, what=f"mixed launch {sh} bits={bits} mode={mode}")


def test_many_tensors_in_one_call(sq):
    """700 small tensors of assorted shapes: the descriptor table goes up in several pieces."""
    rng = np.random.default_rng(8)
    pool = [(8, 16, 3, 3), (4, 64, 1, 1), (16, 1, 3, 3), (3, 5, 5, 5), (2, 128, 3, 3), (5, 33, 1, 1), (1, 2048, 1, 1)]
    shapes = [pool[int(rng.integers(0, len(pool)))] for _ in range(700)]
    ws = [(rng.standard_normal(sh) * 0.05).astype(np.float32) for sh in shapes]
    codes, scales = run_batched(sq, ws, 4, 2)
    for i, (w, c, sc) in enumerate(zip(ws, codes, scales)):
        assert_same(c, sc, w, 4, 2, threads=1, what=f"tensor {i} {w.shape}")


def test_caller_stream_is_honoured(sq):
    """Work goes to the stream handed in: queued behind a long copy on that stream, the result is
    complete once that stream is synchronised, and two streams do not disturb each other."""
    w1 = rand_weights((64, 256, 3, 3), 31, "normal")
    w2 = rand_weights((48, 1024, 1, 1), 32, "heavy")
    d1, d2 = torch.from_numpy(w1).cuda(), torch.from_numpy(w2).cuda()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    big = torch.empty(1 << 26, device="cuda")
    with torch.cuda.stream(s1):
        big.normal_()                                   # keeps s1 busy first
        c1, sc1 = sq.squant_quantize(d1, 4, 2, stream=s1)
    with torch.cuda.stream(s2):
        c2, sc2 = sq.squant_quantize(d2, 8, 2, stream=s2)
    s1.synchronize()
    s2.synchronize()
    assert_same(c1, sc1, w1, 4, 2, what="stream 1")
    assert_same(c2, sc2, w2, 8, 2, what="stream 2")


def test_batched_call_in_a_hip_graph(sq):
    """The calls only enqueue kernels (no allocation, no host synchronisation, no memset), so a
    caller can capture them into a graph.  Replays with new weights in the same buffers, with
    eager work and synchronisations in between, must each match the reference."""
    shapes = [(32, 64, 3, 3), (16, 256, 1, 1), (8, 1, 3, 3), (4, 3, 7, 7), (24, 512, 3, 3), (6, 1028, 1, 1)]
    dws = [torch.zeros(sh, device="cuda") for sh in shapes]
    plan = sq.BatchPlan(dws)
    plan.run(4, 2)                                   # warm-up outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.run(4, 2)
    for rep in range(4):
        ws = [rand_weights(sh, 1000 + 10 * rep + i, "heavy" if (rep + i) % 2 else "normal")
              for i, sh in enumerate(shapes)]
        for d, w in zip(dws, ws):
            d.copy_(torch.from_numpy(w))
        eager = sq.squant_quantize(dws[0], 4, 2)     # the program's own eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for w, c, sc in zip(ws, plan.codes, plan.scales):
            assert_same(c, sc, w, 4, 2, what=f"graph replay {rep} {w.shape}")
        assert torch.equal(eager[0], plan.codes[0])


def test_config5_slice_batched(sq):
    specs = synth.config_specs(5, n_tensors=6)
    ws = [synth.generate(s) for s in specs]
    codes, scales = run_batched(sq, ws, 4, 2)
    for s, w, c, sc in zip(specs, ws, codes, scales):
        assert_same(c, sc, w, 4, 2, what=f"config 5 tensor {s.index} {s.dist}")


def test_config5_full_size_every_tensor(sq):
    """All 256 tensors in one batched call (the benchmark's launch configuration), and every one
    of them compared with the reference in full (it takes the 604 M weights in a few seconds on
    16 threads)."""
    specs = synth.config_specs(5)
    shape = specs[0].shape
    host = [synth.generate(s) for s in specs]
    plan = sq.BatchPlan([torch.from_numpy(w).cuda() for w in host])
    codes, scales = plan.run(4, 2)
    torch.cuda.synchronize()
    for s in specs:
        assert_same(codes[s.index], scales[s.index], host[s.index], 4, 2, threads=16, what=f"C5 tensor {s.index}")
    host_keep = {t: host[t] for t in (0, 129, 255)}
    sample_tensors = sorted(host_keep)
    # properties that hold at any size: codes in range, every scale positive
    for t in (7, 100, 200):
        assert int(codes[t].abs().max()) <= 7
        assert bool((scales[t] > 0).all())
    # Eq. 6-8 recomputed in float64 from (weights, GPU codes, GPU scales) on whole tensors: every
    # channel's perturbation sum within 0.5, every kernel's within 1.0, every element within one
    # step of its quotient (the slack covers the binary32 division and the Q23 grid)
    for t in sorted(sample_tensors):
        w = host_keep[t].astype(np.float64)
        c = codes[t].cpu().numpy().astype(np.float64)
        s = scales[t].cpu().numpy().astype(np.float64)[:, None, None, None]
        p = (c - w / s).reshape(shape[0], shape[1], -1)
        eps = 2.0 ** -17
        assert np.abs(p.sum((-1, -2))).max() <= 0.5 + shape[1] * 9 * eps
        assert np.abs(p.sum(-1)).max() <= 1.0 + 9 * eps
        assert np.abs(p).max() < 1.0 + eps


@pytest.mark.parametrize("kind", ["normal", "heavy", "grid"])
@pytest.mark.parametrize("cout", [1, 63, 64, 65, 960, 4097])
def test_depthwise_3x3_thread_per_channel(sq, cout, kind):
    """Depthwise 3x3 layers: every thread solves a whole output channel."""
    w = rand_weights((cout, 1, 3, 3), 600 + cout, kind)
    if cout > 2:
        w[1] = 0.0
        w[2] = -0.7                      # one-sided: the E&C candidate must flip
    for bits, mode in ((4, 2), (4, 3), (8, 1), (2, 3), (3, 0)):
        codes, scales = run_single(sq, w, bits, mode)
        assert_same(codes, scales, w, bits, mode, what=f"depthwise cout={cout} {kind} bits={bits} mode={mode}")


@pytest.mark.parametrize("shape", [(3, 492, 3, 3), (2, 512, 3, 3), (2, 8192, 1, 1), (2, 32768, 1, 1), (3, 64, 3, 3)])
def test_one_sided_perturbations_have_huge_channel_sums(sq, shape):
    """Every element rounds the same way, so the channel sum reaches thousands of steps: the
    sums must not wrap, and more flips are wanted than there are candidates."""
    w = np.full(shape, -1.25, np.float32)
    w.reshape(shape[0], -1)[:, 0] = 5.0
    w[0].reshape(-1)[3::11] = 0.61
    for bits, mode in ((5, 3), (5, 2), (4, 3), (8, 2), (3, 1)):
        codes, scales = run_single(sq, w, bits, mode)
        assert_same(codes, scales, w, bits, mode, what=f"one-sided {shape} bits={bits} mode={mode}")


# ---------------------------------------------------------------------------
# very long 1x1 / FC channels: held in one workgroup up to cin 65536, the streaming 1x1 kernel beyond
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("kind", ["normal", "heavy", "grid"])
@pytest.mark.parametrize("shape", [(3, 32772, 1, 1), (2, 40000, 1, 1), (2, 65536, 1, 1), (1, 131072, 1, 1),
                                   (2, 65540, 1, 1), (2, 70000, 1, 1)])
def test_streaming_kernel_for_long_channels(sq, shape, kind):
    w = rand_weights(shape, 900 + shape[1] % 97, kind)
    if kind == "normal":
        w[0, 5::7] = 0.0          # plenty of exact zeros next to the small positive perturbations
    for bits, mode in ((4, 2), (8, 2), (3, 0), (2, 3)):
        codes, scales = run_single(sq, w, bits, mode)
        assert_same(codes, scales, w, bits, mode, what=f"stream {shape} {kind} bits={bits} mode={mode}")


@pytest.mark.parametrize("n", [36000, 65540, 70000])
def test_streaming_kernel_degenerate_channels(sq, n):
    """Channels whose perturbations are all equal, all zero, or all on one side (36000: the kernel that holds
    the row in one workgroup)."""
    rows = [np.full(n, 0.3, np.float32), np.zeros(n, np.float32), np.full(n, -1.0, np.float32)]
    half = np.full(n, 2.5, np.float32); half[0] = 7.0            # x = 2.5 everywhere: exact halves
    tiny = np.full(n, 0.01, np.float32); tiny[0] = 7.0           # every element rounds to 0, p < 0 ... same sign
    third = np.full(n, 7.0 / 3.0, np.float32); third[0] = 7.0
    w = np.stack(rows + [half, tiny, third])[:, :, None, None]
    for bits in (4, 8):
        codes, scales = run_single(sq, w, bits, 2)
        assert_same(codes, scales, w, bits, 2, what=f"stream degenerate bits={bits}")


def test_no_channel_is_too_large(sq):
    """Beyond what the on-chip kernels hold, the streaming kernel takes over (see test_gpu_stream.py)."""
    assert sq.squant_max_channel_elems(1, 1) == 1 << 30
    assert sq.squant_max_channel_elems(3, 3) == 1 << 30
    assert sq.squant_max_channel_elems(0, 3) == 0


# ---------------------------------------------------------------------------
# 1x1 / FC widths that take each number of 16-byte vectors per thread (1..8), with full and
# ragged last rounds
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("kind", ["normal", "heavy", "grid"])
@pytest.mark.parametrize("cin", [260, 300, 576, 768, 772, 1280, 1536, 1600, 2560, 4100, 4608, 5120, 5376, 6656,
                                 7168, 7172, 8188])
def test_fc_widths_for_every_vector_count(sq, cin, kind):
    w = rand_weights((3, cin, 1, 1), 900 + cin, kind)
    for bits, mode in ((4, 2), (8, 2), (3, 0)):
        codes, scales = run_single(sq, w, bits, mode)
        assert_same(codes, scales, w, bits, mode, what=f"cin={cin} {kind} bits={bits} mode={mode}")


def test_many_output_channels(sq):
    """A vocabulary-sized FC layer and a wide 1x3 layer: tens of thousands of workgroups per tensor."""
    for shape in ((50257, 768, 1, 1), (30000, 96, 1, 3)):
        w = rand_weights(shape, 61, "normal")
        codes, scales = run_single(sq, w, 4, 2)
        assert_same(codes, scales, w, 4, 2, threads=16, what=f"{shape}")


def test_wave_kernel_walks_several_channels(sq):
    """1x1 / FC channels that take a wave each, in launches of more than 65536 channels: there a
    wave walks four consecutive channels and requests the next one's weights early.  A single
    tensor with a ragged channel count, and a batch of tensors of another width (seven vectors
    per lane, the last one ragged) in all three value distributions."""
    w = rand_weights((70001, 512, 1, 1), 71, "normal")
    codes, scales = run_single(sq, w, 4, 2)
    assert_same(codes, scales, w, 4, 2, threads=16, what="70001 x 512")
    del w, codes, scales
    kinds = ("normal", "heavy", "grid")
    ws = [rand_weights((3001, 1540, 1, 1), 500 + i, kinds[i % 3]) for i in range(24)]
    for bits, mode in ((4, 2), (8, 0)):
        codes, scales = run_batched(sq, ws, bits, mode)
        for i in (0, 1, 2, 13, 23):
            assert_same(codes[i], scales[i], ws[i], bits, mode, threads=16, what=f"tensor {i} of 24 x [3001,1540] {kinds[i % 3]}")
        rng = np.random.default_rng(3)
        for i in range(24):
            for c in rng.integers(0, 3001, 4):
                want_c, want_s = oracle.quantize(ws[i][c][None], bits, mode)
                assert np.array_equal(codes[i][c].cpu().numpy().reshape(-1), want_c.reshape(-1)), f"tensor {i} channel {c}"
                assert scales[i][c].cpu().numpy().view(np.uint32) == want_s.view(np.uint32)[0]
