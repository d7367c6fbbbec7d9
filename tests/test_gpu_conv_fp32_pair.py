"""XNOR_ALGO_MFMA_SPLIT of xnor_conv2d_fp32_fwd_ws in layers of many terms, where both operands are two f16 terms: against the
oracle at the edges of its tiles, rings and chains, and against 64-bit sums beside the form with three terms, which runs
with a workspace one byte short of what the pairs take."""
import zlib

import numpy as np
import pytest
import torch

import oracle
from paper_2007_14178_amd.workloads import random_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xb():
    from paper_2007_14178_amd import binding
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def run(xb, I, Wt, s, pairs=True):
    nbytes = xb.xnor_conv2d_fp32_pairs_workspace_bytes(s)
    assert nbytes > xb.xnor_conv2d_fp32_workspace_bytes(s, xb.ALGO_MFMA_SPLIT) > 0
    ws = torch.full((nbytes - (not pairs),), 0xff, dtype=torch.uint8, device="cuda")
    out = torch.full((s.N, s.F, *xb.xnor_out_dim(s)), float("nan"), device="cuda")
    xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, out, algo=xb.ALGO_MFMA_SPLIT, workspace=ws)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def sums64(I, Wt, s):
    d = [torch.from_numpy(np.ascontiguousarray(a)).double() for a in (I, Wt)]
    return [torch.nn.functional.conv2d(*x, stride=(s.sh, s.sw), padding=(s.ph, s.pw)).numpy() for x in (d, [v.abs() for v in d])]


#        N   C   H   W   F  kh kw sh sw ph pw
SHAPES = [
    (2, 273, 9, 11, 33, 3, 3, 1, 1, 1, 1),       # one channel past a chunk, one filter past a tile, one granule a thread
    (1, 288, 13, 13, 65, 3, 3, 1, 1, 1, 1),      # one filter past a wave
    (1, 1040, 6, 7, 130, 3, 3, 1, 1, 1, 1),      # 65 chunks: the powers of two of more than 64
    (2, 97, 56, 57, 130, 5, 5, 1, 1, 2, 2),      # chains of 10, 10 and 5 taps, the ring of two turned, two granules
    (1, 289, 6, 500, 20, 3, 3, 1, 1, 1, 1),      # rows far wider than a workgroup's pixels
    (2, 300, 31, 29, 70, 3, 3, 2, 2, 1, 1),      # strides
    (1, 640, 9, 9, 12, 2, 2, 1, 1, 1, 1),        # four taps: the commit is longer than the steps
    (1, 176, 12, 14, 40, 3, 5, 1, 2, 1, 2),      # 15 taps: chains of 9 and 6
    (1, 520, 11, 10, 40, 1, 5, 1, 1, 0, 2),      # five taps, the ring of two turned
    (1, 290, 67, 49, 72, 3, 3, 4, 4, 1, 1),      # three granules
    (2, 110, 40, 41, 100, 5, 5, 2, 2, 2, 2),     # three granules and the ring of two
    (8, 288, 28, 28, 264, 3, 3, 1, 1, 1, 1),     # two tiles a wave, a workgroup whose second filter half is short
    (1, 288, 5, 5, 8, 3, 3, 1, 1, 4, 4),         # windows that are all padding
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pair_shapes_vs_oracle(xb, shape):
    print(f"case conv_fp32 pair shape={shape}", flush=True)
    rng = np.random.default_rng(zlib.crc32(("pair" + str(shape)).encode()))
    _, I, Wt = random_layer(rng, "t", *shape)
    O, S = oracle.conv_fp32(I, Wt, oracle.Shape(*shape), want_scale=True)
    err = np.abs(run(xb, I, Wt, xb.Shape(*shape)) - O.astype(np.float64))
    assert (err <= 1e-5 * S).all()
    assert np.sqrt((err ** 2).mean()) <= 2e-7 * np.sqrt((S ** 2).mean()) + 1e-30


@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("shape", [(1, 512, 14, 14, 64, 3), (2, 288, 20, 21, 40, 3), (2, 112, 15, 14, 70, 5), (1, 256, 13, 13, 64, 5)],
                         ids=lambda s: "x".join(map(str, s)))
def test_pairs_are_no_less_exact_than_three_terms(xb, shape, positive):
    """Error against 64-bit sums, on the same data: 0.64 to 0.97 of that of six products (normal values; 0.5 to 0.7 positive)."""
    N, C, H, W, F, k = shape
    print(f"case conv_fp32 pair exactness shape={shape} positive={positive}", flush=True)
    rng = np.random.default_rng(zlib.crc32(str(shape).encode()))
    I, Wt = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((F, C, k, k)).astype(np.float32)
    if positive:
        I, Wt = np.maximum(I, 0), np.abs(Wt)
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, k // 2, k // 2)
    ref, _ = sums64(I, Wt, s)
    pair, three = (np.sqrt(((run(xb, I, Wt, s, p) - ref) ** 2).mean()) for p in (True, False))
    assert 0 < pair <= three, (pair, three)


WHAT = ["tiny corner", "tiny channels", "decayed filter", "decayed weights", "large later", "zeros", "all tiny", "one size up", "log-normal", "subnormal"]


@pytest.mark.parametrize("what", WHAT)
@pytest.mark.parametrize("shape", [(2, 290, 11, 12, 70, 3), (1, 100, 21, 20, 130, 5)], ids=lambda s: "x".join(map(str, s)))
def test_pair_values_of_very_different_sizes(xb, shape, what):
    """What a pair does not hold: regions, channels, filters and single values far from the largest beside them.  The bar is that
    of the fp32 kernels, 1e-5 of S = sum |I * Wt| for every output, where nothing but the far values may be under the window,
    and below fp32's normal range a spacing of 2^-149 a term."""
    N, C, H, W, F, k = shape
    print(f"case conv_fp32 pair sizes shape={shape} {what}", flush=True)
    rng = np.random.default_rng(zlib.crc32((what + str(shape)).encode()))
    I, Wt = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((F, C, k, k)).astype(np.float32)
    if what == "tiny corner":           # windows of values of 2^-30 of the others in their workgroup
        I[:, :, : k + 1, : k + 1] *= np.float32(2.0 ** -30)
    if what == "tiny channels":         # a chunk's channels of very different sizes, and the other way round in the filters
        size = np.float32(2.0) ** -(np.arange(C) % 40).astype(np.float32)
        I *= size[None, :, None, None]
        Wt /= size[None, :, None, None]
    if what == "decayed filter":
        Wt[3] *= np.float32(1e-11)
        Wt[F - 1] = 0
    if what == "decayed weights":       # in one filter and chunk; only those meet values
        Wt[5, :16] *= np.float32(1e-9)
        I[:, 16:, H // 2:] = 0
    if what == "large later":
        I[:, C - 2, 2, 3] = 1e9
    if what == "zeros":
        I[:, :, H // 2:] = 0
        I[0, 0, H - 1, W - 1] = 1e-12
    if what == "all tiny":
        I *= np.float32(1e-30)
    if what == "one size up":           # outputs beyond fp32's largest meet outputs within
        I *= np.float32(1e19)
        Wt[: F // 2] *= np.float32(1e18)
    if what == "log-normal":
        I = np.exp(4 * rng.standard_normal(I.shape)).astype(np.float32)
    if what == "subnormal":
        I[:, :, :4] = np.float32(1e-40)
        Wt[1] *= np.float32(1e-38)
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, k // 2, k // 2)
    got = run(xb, I, Wt, s)
    ref, S = sums64(I, Wt, s)
    held = np.abs(ref) < 3.4e38
    if what == "one size up":
        assert not np.isfinite(got[np.abs(ref) > 3.5e38]).any() and held[:, F // 2:].all() and not held.all()
        held &= S < 3.4e38              # (a partial sum may leave the range where the whole does not)
    assert (np.abs(got - ref)[held] <= 1e-5 * S[held] + C * k * k * 2.0 ** -149).all()


@pytest.mark.parametrize("k", [3, 5])
def test_pair_outputs_formed_one_by_one(xb, k):
    """A few outputs whose windows hold zeros, or one value far below the others, in a workgroup with values that pairs do not
    hold: three filters, so that a wave has no more than it forms one by one."""
    C = 290 if k == 3 else 100
    print(f"case conv_fp32 pair few k={k}", flush=True)
    rng = np.random.default_rng(3)
    I, Wt = rng.standard_normal((2, C, 16, 16)).astype(np.float32), rng.standard_normal((3, C, k, k)).astype(np.float32)
    I[0, 7, 1, 1] = 3e-9
    I[0, :, 8:8 + k, 8:8 + k] = 0                # one window of nothing
    I[1, :, 8:8 + k, 8:8 + k] = 0
    I[1, C - 1, 9, 9] = 1e-9                     # one of a single value
    s = xb.Shape(2, C, 16, 16, 3, k, k, 1, 1, k // 2, k // 2)
    got = run(xb, I, Wt, s)
    ref, S = sums64(I, Wt, s)
    assert (np.abs(got - ref) <= 1e-5 * S).all()
    c = 8 + k // 2
    assert (got[0, :, c, c] == 0).all() and (np.abs(got[1, :, c, c] / ref[1, :, c, c] - 1) <= 2.0 ** -23).all()


@pytest.mark.parametrize("k", [3, 5])
def test_pair_inputs_that_are_not_finite(xb, k):
    """Infinities, NaN and values at the top of the range, in input and weights, give what one thread per output gives."""
    N, C, H, W, F = 1, 290 if k == 3 else 100, 20, 20, 70
    print(f"case conv_fp32 pair not finite k={k}", flush=True)
    rng = np.random.default_rng(5)
    I, Wt = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((F, C, k, k)).astype(np.float32)
    I[0, 3, 2, 2], I[0, 70, 17, 17], I[0, 5, 17, 2], I[0, 7, 2, 17] = np.inf, -np.inf, np.nan, 3.4028235e38
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, 1, 1)
    for weights in (False, True):
        if weights:
            I = np.where(np.isfinite(I) & (np.abs(I) < 1e30), I, 0).astype(np.float32)
            Wt[1, C - 1, 0, 0], Wt[2, 0, k - 1, 0], Wt[3, 1, 1, 1], Wt[33, 2, 0, 0] = np.inf, -np.inf, np.nan, 3.402e38
        ref = xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, algo=xb.ALGO_DIRECT).cpu().numpy().astype(np.float64)
        got = run(xb, I, Wt, s)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).any()
        assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.isinf(ref).any()
        assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
        fine = np.isfinite(ref)
        _, S = sums64(np.where(np.isfinite(I), I, 0), np.where(np.isfinite(Wt), Wt, 0), s)
        assert (np.abs(got[fine] - ref[fine]) <= 1e-5 * S[fine]).all()


def test_pair_in_a_graph(xb):
    """Captured and replayed on other values in the same buffers, eager work between the replays."""
    N, C, H, W, F, k = 4, 288, 20, 20, 96, 3
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, 1, 1)
    g = torch.Generator(device="cuda").manual_seed(2)
    I, Wt = torch.randn((N, C, H, W), generator=g, device="cuda"), torch.randn((F, C, k, k), generator=g, device="cuda")
    ws = torch.empty((xb.xnor_conv2d_fp32_pairs_workspace_bytes(s),), dtype=torch.uint8, device="cuda")
    out = torch.empty((N, F, H, W), device="cuda")
    xb.xnor_conv2d_fp32_fwd(I, Wt, s, out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        xb.xnor_conv2d_fp32_fwd(I, Wt, s, out, workspace=ws)
    for i in range(3):
        I.copy_(torch.randn(I.shape, generator=g, device="cuda"))
        if i == 1:
            I[0, :, :8] *= 1e-9
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, xb.xnor_conv2d_fp32_fwd(I, Wt, s))


def test_pairs_by_the_workspace_and_the_number_of_terms(xb):
    """Two terms from 160 (tap, chunk) steps on and with their workspace, three below and with a smaller one."""
    for C, k, pairs in ((288, 3, True), (272, 3, False), (512, 1, False), (2576, 1, False), (97, 5, True), (96, 5, False), (640, 2, True), (64, 7, False)):
        assert (xb.xnor_conv2d_fp32_pairs_workspace_bytes(xb.Shape(1, C, 12, 12, 40, k, k, 1, 1, k // 2, k // 2)) > 0) == pairs, (C, k)
    s = xb.Shape(1, 288, 12, 12, 40, 3, 3, 1, 1, 1, 1)
    rng = np.random.default_rng(1)
    I, Wt = rng.standard_normal((1, 288, 12, 12)).astype(np.float32), rng.standard_normal((40, 288, 3, 3)).astype(np.float32)
    pair, three = run(xb, I, Wt, s), run(xb, I, Wt, s, False)
    assert not np.array_equal(pair, three)
    assert np.array_equal(pair, xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s).cpu().numpy())
    ws = torch.empty((xb.xnor_conv2d_fp32_workspace_bytes(s),), dtype=torch.uint8, device="cuda")
    assert np.array_equal(three, xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, workspace=ws).cpu().numpy())


@pytest.mark.parametrize("what", ["values", "one value", "channels", "equal"])
@pytest.mark.parametrize("p", [12, 17, 19, 20, 22])
@pytest.mark.parametrize("shape", [(1, 512, 13, 13, 64, 3), (1, 256, 17, 17, 70, 5)], ids=lambda s: "x".join(map(str, s)))
def test_pairs_beside_larger_values_are_no_less_exact_than_three_terms(xb, shape, p, what):
    """Values of 2^-p of others in their workgroup's chunk, values of different mantissas or all of one (what a pair loses of that
    adds up).  Error over the outputs whose windows hold none of the larger ones, against what their terms' sizes make a sum's
    rounding, of both forms on the same data: 0.76 to 0.95 of that of three terms."""
    N, C, H, W, F, k = shape
    print(f"case conv_fp32 pair beside larger shape={shape} p={p} {what}", flush=True)
    rng = np.random.default_rng(zlib.crc32((what + str(p) + str(shape)).encode()))
    I, Wt = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((F, C, k, k)).astype(np.float32)
    far = np.zeros((N, C, H, W), bool)
    far[:, ::16, 4::8, 4::8] = True
    if what == "values":
        I = np.sign(I) * (1 + rng.random(I.shape)).astype(np.float32)
    if what == "one value":
        I = np.where(I < 0, np.float32(-0.6663), np.float32(1.3337))
    if what == "channels":              # of a chunk, beside the larger values too
        I *= (np.float32(2.0) ** -(np.arange(C) % 16).astype(np.float32))[None, :, None, None]
    if what == "equal":
        I, Wt = np.full_like(I, 1.3337), np.broadcast_to((1 + rng.random((F, 1, 1, 1))).astype(np.float32), Wt.shape).copy()
    I[far] = np.float32(2.0) ** p
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, k // 2, k // 2)
    ref, _ = sums64(I, Wt, s)
    size = np.sqrt(sums64(I.astype(np.float64) ** 2, Wt.astype(np.float64) ** 2, s)[0])
    clear = sums64(far.astype(np.float32), np.ones_like(Wt), s)[0] == 0
    assert clear.any() and not clear.all()
    pair, three = (np.sqrt((((run(xb, I, Wt, s, f) - ref) / size)[clear] ** 2).mean()) for f in (True, False))
    assert 0 < pair <= three, (pair, three)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_pairs_run_by_name_and_by_workspace(xb, shape):
    """Values of one size are summed from pairs in every workgroup (another form would give that form's bits), and either form has
    a name under which the size of the workspace makes no difference."""
    print(f"case conv_fp32 pair forms shape={shape}", flush=True)
    rng = np.random.default_rng(zlib.crc32(("forms" + str(shape)).encode()))
    s = xb.Shape(*shape)
    I, Wt = ((1 + rng.random(d)) * rng.choice([-1, 1], d) for d in ((s.N, s.C, s.H, s.W), (s.F, s.C, s.kh, s.kw)))
    I, Wt = dev(I.astype(np.float32)), dev(Wt.astype(np.float32))
    small, large = xb.xnor_conv2d_fp32_workspace_bytes(s, xb.ALGO_MFMA_SPLIT_THREE), xb.xnor_conv2d_fp32_workspace_bytes(s, xb.ALGO_MFMA_SPLIT_PAIRS)
    assert large == xb.xnor_conv2d_fp32_pairs_workspace_bytes(s) > small == xb.xnor_conv2d_fp32_workspace_bytes(s, xb.ALGO_MFMA_SPLIT)

    def form(algo, nbytes):
        return xb.xnor_conv2d_fp32_fwd(I, Wt, s, algo=algo, workspace=torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda"))

    pairs, three = form(xb.ALGO_MFMA_SPLIT_PAIRS, large), form(xb.ALGO_MFMA_SPLIT_THREE, small)
    ref, S = sums64(I.cpu().numpy(), Wt.cpu().numpy(), s)
    # (an output of a few terms, at a corner, can have the same bits either way; most of a 32 x 32 tile's can not)
    differ = (pairs != three).cpu().numpy()[S > 0]
    assert differ.mean() > 0.25
    assert torch.equal(form(xb.ALGO_MFMA_SPLIT_THREE, 2 * large), three) and torch.equal(form(xb.ALGO_MFMA_SPLIT, large - 1), three)
    assert torch.equal(form(xb.ALGO_MFMA_SPLIT_PAIRS, 2 * large), pairs) and torch.equal(form(xb.ALGO_MFMA_SPLIT, large), pairs)
    for algo, want in ((xb.ALGO_MFMA_SPLIT_PAIRS, pairs), (xb.ALGO_MFMA_SPLIT_THREE, three)):
        assert torch.equal(xb.xnor_conv2d_fp32_fwd(I, Wt, s, algo=algo), want)
