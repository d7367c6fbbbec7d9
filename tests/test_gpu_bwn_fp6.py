"""The FP6 form of xnor_bwn_conv2d_fwd (five E2M3 digits per input value, one scale per position and 32 channels)
against 64-bit sums, at the edges of its tiles, chunks and scales, and the form it leaves some shapes to.

Bars.  Held digits: a value is off by at most 2^-22 of its block's scale, which is at most 2^-23.9 of the block's largest
value, so an output by at most 32 * 2^-23.9 < 2.1e-6 of alpha * S (S = the sum of magnitudes under the window): inside the
1e-5 that all kernels of the call are held to, in the worst case.  Beside it 2^-125 per value, the documented floor."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xb():
    from paper_2007_14178_amd import binding
    return binding


def sums64(I, Wt, s):
    """The convolution of I with the filters' signs, and of |I| with ones, in 64 bits on the CPU."""
    x = torch.nn.functional.pad(I.double(), (s.pw, s.pw, s.ph, s.ph))
    sign = torch.where(Wt >= 0, 1.0, -1.0).double()
    cols = torch.nn.functional.unfold(x, (s.kh, s.kw), stride=(s.sh, s.sw))
    OH, OW = (s.H + 2 * s.ph - s.kh) // s.sh + 1, (s.W + 2 * s.pw - s.kw) // s.sw + 1
    out = torch.matmul(sign.reshape(s.F, -1), cols)
    return out.reshape(s.N, s.F, OH, OW), cols.abs().sum(1).reshape(s.N, 1, OH, OW)


def run(xb, shape, I, seed, algo=None):
    print(f"case bwn-fp6 shape={shape} seed={seed}", flush=True)
    s = xb.Shape(*shape)
    Wt = torch.randn((s.F, s.C, s.kh, s.kw), generator=torch.Generator().manual_seed(seed + 1)) * 0.05
    Wpk, alpha, _ = xb.xnor_filter_prepare(Wt.cuda())
    OH, OW = (s.H + 2 * s.ph - s.kh) // s.sh + 1, (s.W + 2 * s.pw - s.kw) // s.sw + 1
    out = torch.full((s.N, s.F, OH, OW), float("nan"), device="cuda")
    xb.xnor_bwn_conv2d_fwd(I.cuda(), Wpk, alpha, s, out=out, algo=algo or xb.ALGO_MFMA_SPLIT_FP6)
    torch.cuda.synchronize()
    return out.cpu().double(), alpha.cpu().double()[None, :, None, None], *sums64(I, Wt, s), s


def check(xb, shape, I, seed, algo=None):
    got, alpha, ref, S, s = run(xb, shape, I, seed, algo)
    bar = alpha * (1e-5 * S + s.C * s.kh * s.kw * 2.0 ** -125)
    err = (got - alpha * ref).abs()
    assert bool((err <= bar).all()), f"worst err/bar {float((err / bar.clamp_min(1e-300)).nan_to_num(1e9).max()):.3g}"
    assert float(err.pow(2).mean().sqrt()) <= 2e-7 * float((alpha * S).pow(2).mean().sqrt()) + 1e-30


#        N   C   H   W    F  kh kw sh sw ph pw
SHAPES = [
    (1, 1, 1, 1, 1, 1, 1, 1, 1, 0, 0),
    (2, 32, 4, 8, 32, 1, 1, 1, 1, 0, 0),         # one tile exactly; one word, one tap: half a step
    (2, 33, 3, 11, 33, 2, 1, 1, 1, 0, 0),        # a second word of one channel; an even number of taps
    (3, 64, 31, 1, 31, 3, 3, 1, 1, 1, 1),        # rows one value wide, 31 pixels
    (1, 65, 11, 3, 65, 3, 3, 1, 1, 1, 1),        # two chunks, the last one of one word
    (2, 96, 13, 13, 97, 3, 3, 1, 1, 1, 1),
    (1, 127, 9, 29, 128, 5, 3, 2, 1, 2, 1),
    (2, 160, 16, 16, 129, 3, 3, 1, 1, 1, 1),     # 8 tiles
    (1, 64, 17, 16, 40, 3, 3, 1, 1, 1, 1),       # 8 tiles and 16 pixels
    (2, 40, 9, 9, 4, 3, 3, 1, 1, 5, 4),          # windows that are all padding
    (1, 70, 15, 17, 130, 1, 7, 1, 3, 0, 3),
    (1, 48, 20, 34, 70, 8, 8, 1, 2, 3, 3),       # 64 taps
    (16, 128, 56, 56, 128, 3, 3, 1, 1, 1, 1),    # four filter tiles a wave
    (64, 96, 14, 14, 96, 3, 3, 1, 1, 1, 1),
    (64, 96, 14, 14, 256, 3, 3, 1, 1, 1, 1),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_tiles_and_chunks(xb, shape):
    g = torch.Generator().manual_seed(sum(shape))
    check(xb, shape, torch.randn(shape[:4], generator=g), sum(shape))


def test_every_sum_of_24_bit_integers_is_exact(xb):
    """Values of up to 24 bits in the block's top binade have no error; few terms, so the sums have none either."""
    shape = (1, 32, 6, 9, 33, 1, 1, 1, 1, 0, 0)
    g = torch.Generator().manual_seed(3)
    I = torch.zeros(shape[:4])
    at = torch.randint(0, 32, (6, 9), generator=g)
    for y in range(6):
        for x in range(9):
            I[0, at[y, x], y, x] = float(2 ** 23 + int(torch.randint(0, 2 ** 23, (1,), generator=g))) * 2.0 ** (3 * (x - 4)) * (-1) ** y
    got, alpha, ref, _, _ = run(xb, shape, I, 3)
    assert torch.equal(got, (ref.float() * alpha.float()).double())


@pytest.mark.parametrize("top", [1.9374999, 1.9375, 1.9375001, 1.9999999, 1.0, 1.5])
def test_scales_around_the_largest_digit(xb, top):
    """The block's largest value on either side of where the scale steps, over fp32's exponents from the smallest up to 2^121."""
    shape = (1, 64, 9, 28, 36, 1, 1, 1, 1, 0, 0)
    g = torch.Generator().manual_seed(5)
    I = (torch.rand(shape[:4], generator=g) * 2 - 1).numpy().astype(np.float32)
    I[0, 7] = np.float32(top)
    I[0, 40] = -np.float32(top)
    power = np.arange(252).reshape(9, 28) - 126
    I = np.ldexp(I, power[None, None] - 5 * (power > 118)).astype(np.float32)
    got, alpha, ref, S, s = run(xb, shape, torch.from_numpy(I), 5)
    err = (got - alpha * ref).abs()
    assert bool((err <= alpha * (1e-5 * S + s.C * 2.0 ** -125) + 2.0 ** -149).all())


@pytest.mark.parametrize("top", [1.875, 1.9374999, 1.9375, 1.96875, float(np.finfo(np.float32).max) / 2.0 ** 127], ids=lambda v: f"{v:.7f}")
@pytest.mark.parametrize("form", ["FP6", "BF16"])
@pytest.mark.parametrize("shape", [(1, 1, 9, 28, 36, 1, 1, 1, 1, 0, 0), (2, 70, 12, 12, 40, 1, 1, 1, 1, 0, 0), (1, 40, 9, 12, 100, 3, 3, 1, 1, 1, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_values_at_the_top_of_the_range(xb, shape, top, form):
    """One value of up to the largest float under a window, of either sign, others of its block small or zero: the sums are
    inside fp32's range, so they are finite and inside the bar (filters of 0.05 keep the outputs in range too)."""
    g = torch.Generator().manual_seed(7)
    I = torch.randn(shape[:4], generator=g) * 2.0 ** torch.randint(-20, 100, (shape[0], 1, *shape[2:4]), generator=g)
    I[:, :, ::2] = 0
    for k, (y, x) in enumerate(((1, 1), (1, 5), (4, 1), (4, 9), (7, 4))):
        I[:, :, y - 1:y + 2, x - 1:x + 2] *= 2.0 ** -60
        I[:, (17 * k) % shape[1], y, x] = float(np.float32(top)) * 2.0 ** 127 * (-1) ** k
    check(xb, shape, I, 7, getattr(xb, "ALGO_MFMA_SPLIT_" + form))


def test_small_values_beside_large_ones(xb):
    """Magnitudes of 40 binades within the blocks: the error stays that of the largest value, and a position of small
    values beside one of large ones keeps its own scale."""
    shape = (2, 80, 12, 12, 40, 1, 1, 1, 1, 0, 0)
    g = torch.Generator().manual_seed(9)
    I = torch.randn(shape[:4], generator=g) * torch.exp2(torch.randint(-20, 21, shape[:4], generator=g).float())
    I[:, :, ::2] *= 2.0 ** -30
    check(xb, shape, I, 9)


def test_not_finite_inputs_reach_their_windows_only(xb):
    shape = (2, 70, 12, 14, 37, 3, 3, 1, 1, 1, 1)
    g = torch.Generator().manual_seed(11)
    I = torch.randn(shape[:4], generator=g)
    bad = torch.zeros((2, 1, 12, 14))
    for n, c, y, x, v in ((0, 3, 0, 0, float("nan")), (0, 69, 7, 9, float("inf")), (1, 33, 11, 13, -float("inf"))):
        I[n, c, y, x] = v
        bad[n, 0, y, x] = 1
    got, alpha, _, _, s = run(xb, shape, I, 11)
    hit = torch.nn.functional.max_pool2d(bad, 3, 1, 1).bool().expand_as(got)
    assert bool(torch.isnan(got[hit]).all()) and bool(torch.isfinite(got[~hit]).all())
    check_I = torch.where(torch.isfinite(I), I, torch.zeros(()))
    ref, S = sums64(check_I, torch.randn((s.F, s.C, 3, 3), generator=torch.Generator().manual_seed(12)) * 0.05, s)
    assert bool(((got - alpha * ref).abs()[~hit] <= (alpha * 1e-5 * S)[~hit]).all())


def test_rows_too_wide_for_whole_rows_keep_the_bf16_form(xb):
    """Large strides: 32 output pixels lie on two output rows, with nine input rows of 400 under them."""
    shape = (2, 40, 33, 400, 70, 1, 1, 8, 8, 0, 0)
    assert xb.xnor_bwn_split_kernel(xb.Shape(*shape)) == xb.ALGO_MFMA_SPLIT_BF16
    I = torch.randn(shape[:4], generator=torch.Generator().manual_seed(13))
    with pytest.raises(xb.XnorError):
        check(xb, shape, I, 13)
    check(xb, shape, I, 13, xb.ALGO_MFMA_SPLIT)


def test_captured_launches_replay_the_eager_result(xb):
    shape = (4, 96, 14, 14, 100, 3, 3, 1, 1, 1, 1)
    s = xb.Shape(*shape)
    print(f"case bwn-fp6-graph shape={shape}", flush=True)
    g = torch.Generator().manual_seed(17)
    I, Wt = torch.randn(shape[:4], generator=g).cuda(), torch.randn((100, 96, 3, 3), generator=g).cuda()
    Wpk, alpha, _ = xb.xnor_filter_prepare(Wt)
    out = torch.empty((4, 100, 14, 14), device="cuda")
    assert xb.xnor_bwn_pick_algo(s) == xb.ALGO_MFMA_SPLIT and xb.xnor_bwn_split_kernel(s) == xb.ALGO_MFMA_SPLIT_FP6
    xb.xnor_bwn_conv2d_fwd(I, Wpk, alpha, s, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        xb.xnor_bwn_conv2d_fwd(I, Wpk, alpha, s, out=out)
    for scale in (1.0, -3.0, 0.25):
        I.mul_(scale)
        want = xb.xnor_bwn_conv2d_fwd(I, Wpk, alpha, s).clone()
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


#        N   C   H   W    F  kh kw sh sw ph pw: workgroups with splits and with stagers, and layers beside them that have none
SPLIT_SHAPES = [
    (1, 256, 14, 14, 256, 3, 3, 1, 1, 1, 1),     # stagers, one filter tile a wave
    (2, 271, 13, 14, 250, 3, 3, 1, 1, 1, 1),     # ... a last word of 15 channels, an odd number of chunks, a short last tile
    (32, 512, 7, 7, 505, 3, 3, 1, 1, 1, 1),      # ... two splits, the last one's filters short
    (3, 97, 12, 12, 33, 3, 3, 1, 1, 1, 1),       # ... a last filter tile of one filter, a last chunk of one word of one channel
    (2, 448, 5, 6, 32, 3, 3, 1, 1, 1, 1),        # ... fewer pixels than the tiles have
    (8, 192, 27, 27, 256, 5, 5, 1, 1, 2, 2),     # ... several rounds a chunk
    (76, 448, 10, 10, 32, 3, 3, 2, 2, 1, 1),     # ... strides
    (2, 64, 9, 9, 70, 1, 1, 1, 1, 0, 0),         # ... one chunk, one tap
    (4, 320, 9, 70, 64, 1, 1, 2, 2, 0, 0),
    (1, 96, 8, 8, 40, 3, 3, 1, 1, 6, 6),         # ... windows, and workgroups, that are all padding
    (1, 160, 3, 40, 20, 2, 5, 3, 1, 4, 0),
    (128, 384, 13, 13, 384, 3, 3, 1, 1, 1, 1),   # two splits without stagers
    (120, 390, 13, 13, 300, 3, 3, 1, 1, 1, 1),   # neither, beside it: more filters than the splits' estimate takes
]


@pytest.mark.parametrize("shape", SPLIT_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_splits_and_stagers(xb, shape):
    """Sums in a chain of their own per wave, in the order of the chunks' words, whatever the workgroup's shape: the same bars."""
    big = shape[0] > 64
    if big:                                      # (64-bit sums of the first and the last images)
        n = shape[0]
        I = torch.randn(shape[:4], generator=torch.Generator().manual_seed(1))
        I[2:n - 2] = I[:1]
        print(f"case bwn-fp6 splits shape={shape}", flush=True)
        s, one = xb.Shape(*shape), xb.Shape(4, *shape[1:])
        Wt = torch.randn((s.F, s.C, s.kh, s.kw), generator=torch.Generator().manual_seed(2)) * 0.05
        Wpk, alpha, _ = xb.xnor_filter_prepare(Wt.cuda())
        got = xb.xnor_bwn_conv2d_fwd(I.cuda(), Wpk, alpha, s, algo=xb.ALGO_MFMA_SPLIT_FP6).cpu().double()
        at = [0, 1, n - 2, n - 1]
        ref, S = sums64(I[at], Wt, one)
        a = alpha.cpu().double()[None, :, None, None]
        assert torch.equal(got[2:n - 2], got[:1].expand(n - 4, -1, -1, -1))
        assert bool(((got[at] - a * ref).abs() <= a * 1e-5 * S).all())
    else:
        check(xb, shape, torch.randn(shape[:4], generator=torch.Generator().manual_seed(sum(shape))), sum(shape))


@pytest.mark.parametrize("shape", [(1, 256, 14, 14, 256, 3, 3, 1, 1, 1, 1), (128, 384, 13, 13, 384, 3, 3, 1, 1, 1, 1)], ids=lambda s: "x".join(map(str, s)))
def test_splits_and_stagers_in_a_graph(xb, shape):
    """Captured and replayed on new inputs in the same buffers: the eager results each time."""
    print(f"case bwn-fp6 graph shape={shape}", flush=True)
    s = xb.Shape(*shape)
    g = torch.Generator(device="cuda").manual_seed(4)
    I, Wt = torch.randn(shape[:4], generator=g, device="cuda"), torch.randn((s.F, s.C, s.kh, s.kw), generator=g, device="cuda")
    Wpk, alpha, _ = xb.xnor_filter_prepare(Wt)
    out = xb.xnor_bwn_conv2d_fwd(I, Wpk, alpha, s)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        xb.xnor_bwn_conv2d_fwd(I, Wpk, alpha, s, out)
    for _ in range(3):
        I.copy_(torch.randn(shape[:4], generator=g, device="cuda"))
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, xb.xnor_bwn_conv2d_fwd(I, Wpk, alpha, s))


#    N   C   H   W    F  k  s, what the workgroups are: filter tiles a wave, words a chunk, splits, pixel tiles, stagers
FORMS = [
    ((1, 68, 16, 16, 29, 3, 2), (1, 1, 1, 2, 4)),       # three chunks of a word
    ((5, 71, 34, 26, 26, 1, 2), (1, 1, 1, 1, 3)),
    ((1, 100, 5, 5, 32, 1, 1), (1, 2, 1, 1, 3)),
    ((2, 109, 37, 50, 100, 3, 2), (1, 1, 2, 2, 4)),     # several rounds a chunk
    ((14, 61, 36, 36, 90, 7, 2), (1, 1, 3, 1, 4)),      # three splits, the last one's filters short
    ((3, 90, 25, 23, 33, 1, 2), (1, 2, 2, 1, 4)),       # a split of one filter
    ((13, 102, 28, 23, 34, 1, 1), (1, 2, 2, 2, 3)),     # ... of two, two pixel tiles
    ((3, 76, 19, 18, 73, 3, 2), (1, 2, 3, 1, 4)),
    ((1, 43, 16, 22, 297, 3, 2), (1, 2, 3, 1, 4)),      # ... two splits of the last group without filters
    ((2, 51, 25, 25, 112, 3, 2), (1, 2, 4, 1, 4)),      # four splits
    ((10, 190, 27, 27, 486, 3, 2), (2, 1, 3, 1, 4)),    # two filter tiles a wave
    ((28, 62, 33, 26, 213, 3, 2), (2, 1, 4, 1, 4)),     # ... the last split's second tile empty
    ((17, 35, 27, 31, 68, 1, 1), (2, 2, 2, 2, 4)),
    ((21, 52, 17, 17, 205, 1, 1), (2, 2, 2, 2, 3)),
    ((18, 226, 15, 14, 450, 3, 1), (2, 2, 4, 1, 4)),
    ((24, 53, 28, 29, 131, 1, 1), (1, 2, 2, 2, 0)),     # splits without stagers
    ((14, 104, 38, 29, 484, 1, 1), (2, 2, 2, 2, 0)),
    ((19, 126, 35, 48, 137, 3, 1), (3, 1, 2, 2, 0)),    # ... the second split's filters short
    ((24, 74, 36, 36, 134, 3, 1), (3, 2, 2, 2, 0)),
]


@pytest.mark.parametrize("layer, form", FORMS, ids=lambda v: "x".join(map(str, v)))
def test_workgroups_of_every_form(xb, layer, form):
    """The form is what the plan for 256 units says that it is, and the device's plan is that one."""
    N, C, H, W, F, k, st = layer
    shape = (N, C, H, W, F, k, k, st, st, k // 2, k // 2)
    plan = xb.xnor_bwn_fp6_plan(xb.Shape(*shape), 256)
    assert tuple(plan[n] for n in ("filter_tiles", "words", "splits", "tiles", "stagers")) == form
    assert xb.xnor_bwn_fp6_plan(xb.Shape(*shape)) == plan
    check(xb, shape, torch.randn(shape[:4], generator=torch.Generator().manual_seed(sum(shape))), sum(shape))
