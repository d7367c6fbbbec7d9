"""XNOR_ALGO_MFMA_SPLIT of xnor_conv2d_fp32_fwd_ws (both operands as three bf16 terms)
against the oracle, at the edges of its tiles, chunks and dispatch.

The bar against the oracle is that of the fp32 kernels (tests/test_gpu_conv_fp32.py): |got - ref| <=
1e-5 * S with S = sum |I * Wt| over the output's terms, and an RMS error of at most 2e-7 of the RMS of S.
That catches a wrong term, not a lost bit: what the split keeps is held against 64-bit sums below.
"""
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


def split(xb, I, Wt, s):
    ws = torch.empty((16 << 20,), dtype=torch.uint8, device="cuda")
    out = torch.full((s.N, s.F, *xb.xnor_out_dim(s)), float("nan"), device="cuda")
    xb.xnor_conv2d_fp32_fwd(I, Wt, s, out, algo=xb.ALGO_MFMA_SPLIT, workspace=ws)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


#        N   C   H   W   F  kh kw sh sw ph pw
SHAPES = [
    (1, 1, 1, 1, 1, 1, 1, 1, 1, 0, 0),           # one value, one tap, one chunk
    (2, 17, 9, 11, 33, 3, 3, 1, 1, 1, 1),        # one channel past a chunk, one filter past a tile
    (1, 16, 8, 4, 64, 3, 3, 1, 1, 1, 1),         # whole chunk, 32 outputs, one filter wave
    (1, 48, 13, 13, 65, 3, 3, 1, 1, 1, 1),       # 169 outputs, one filter past a wave
    (3, 40, 28, 28, 200, 3, 3, 1, 1, 1, 1),      # six tiles per workgroup, a short last one
    (2, 32, 56, 57, 130, 5, 5, 1, 1, 2, 2),      # two-dimensional tiles, ragged on both sides
    (1, 33, 6, 500, 20, 3, 3, 1, 1, 1, 1),       # rows far wider than a workgroup's pixels
    (2, 24, 31, 29, 70, 3, 5, 2, 3, 1, 2),       # strides, non-square window
    (1, 20, 9, 9, 12, 3, 3, 1, 1, 4, 4),         # windows that are all padding
    (2, 30, 23, 23, 66, 7, 7, 1, 1, 3, 3),       # short chains (49 taps)
    (1, 130, 14, 15, 140, 7, 7, 2, 2, 3, 3),     # short chains, stride, tails everywhere
    (1, 18, 3, 700, 9, 5, 5, 1, 1, 2, 2),        # a row wider than the fp32 matrix kernel stages
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_split_shapes_vs_oracle(xb, shape):
    print(f"case conv_fp32 split shape={shape}", flush=True)
    rng = np.random.default_rng(zlib.crc32(("split" + str(shape)).encode()))
    _, I, Wt = random_layer(rng, "t", *shape)
    O, S = oracle.conv_fp32(I, Wt, oracle.Shape(*shape), want_scale=True)
    err = np.abs(split(xb, dev(I), dev(Wt), xb.Shape(*shape)) - O.astype(np.float64))
    assert (err <= 1e-5 * S).all()
    assert np.sqrt((err ** 2).mean()) <= 2e-7 * np.sqrt((S ** 2).mean()) + 1e-30


@pytest.mark.parametrize("k", [3, 7])
def test_split_inputs_that_are_not_finite(xb, k):
    """Infinities, NaN and values at the top of the range give what the plain fp32 sum gives."""
    shape = (1, 24, 20, 20, 40, k, k, 1, 1, 1, 1)
    print(f"case conv_fp32 split not finite k={k}", flush=True)
    rng = np.random.default_rng(5)
    _, I, Wt = random_layer(rng, "t", *shape)
    I[0, 3, 2, 2], I[0, 20, 17, 17], I[0, 5, 17, 2], I[0, 7, 2, 17] = np.inf, -np.inf, np.nan, 3.4028235e38
    s = xb.Shape(*shape)
    ref = xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, algo=xb.ALGO_DIRECT).cpu().numpy().astype(np.float64)
    got = split(xb, dev(I), dev(Wt), s)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).any()
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.isinf(ref).any()
    fine = np.isfinite(ref)
    assert np.array_equal(np.sign(got[~fine & ~np.isnan(ref)]), np.sign(ref[~fine & ~np.isnan(ref)]))
    S = torch.nn.functional.conv2d(torch.from_numpy(I).double().abs(), torch.from_numpy(Wt).double().abs(), padding=1).numpy()
    with np.errstate(invalid="ignore"):
        assert (np.abs(got - ref)[fine] <= 1e-5 * S[fine]).all()


@pytest.mark.parametrize("scale_I,scale_W", [(2.0 ** -110, 1.0), (1.0, 2.0 ** -112), (2.0 ** -60, 2.0 ** -60), (2.0 ** -100, 2.0 ** 90)])
def test_split_at_the_bottom_of_the_range(xb, scale_I, scale_W):
    """Scaling by powers of two: terms of the split fall below 2^-126 where the fp32 values do not.
    The bar has the roundings of products and partial sums below the normal range beside the 1e-5."""
    shape = (1, 20, 12, 12, 33, 3, 3, 1, 1, 1, 1)
    print(f"case conv_fp32 split tiny {scale_I} {scale_W}", flush=True)
    rng = np.random.default_rng(6)
    I = (rng.standard_normal((1, 20, 12, 12)) * scale_I).astype(np.float32)
    Wt = (rng.standard_normal((33, 20, 3, 3)) * scale_W).astype(np.float32)
    O, S = oracle.conv_fp32(I, Wt, oracle.Shape(*shape), want_scale=True)
    got = split(xb, dev(I), dev(Wt), xb.Shape(*shape))
    assert (np.abs(got - O.astype(np.float64)) <= 1e-5 * S + 2 * 180 * 2.0 ** -149).all()


def test_auto_takes_the_split_kernel_and_refusals_stay(xb):
    s = xb.Shape(2, 40, 20, 20, 72, 3, 3, 1, 1, 1, 1)
    _, I, Wt = random_layer(np.random.default_rng(8), "t", 2, 40, 20, 20, 72, 3, 3, 1, 1, 1, 1)
    I, Wt = dev(I), dev(Wt)
    assert xb.xnor_conv2d_fp32_workspace_bytes(s) > 0
    ws = torch.empty((16 << 20,), dtype=torch.uint8, device="cuda")
    auto = xb.xnor_conv2d_fp32_fwd(I, Wt, s)
    forced = xb.xnor_conv2d_fp32_fwd(I, Wt, s, algo=xb.ALGO_MFMA_SPLIT, workspace=ws)
    plain = xb.xnor_conv2d_fp32_fwd(I, Wt, s, workspace=None)
    mfma = xb.xnor_conv2d_fp32_fwd(I, Wt, s, algo=xb.ALGO_MFMA)
    torch.cuda.synchronize()
    assert torch.equal(auto, forced) and torch.equal(plain, mfma)
    with pytest.raises(xb.XnorError) as e:
        xb.xnor_conv2d_fp32_fwd(I, Wt, s, algo=xb.ALGO_MFMA_SPLIT, workspace=ws[:1024])
    assert e.value.status == xb.E_WORKSPACE
    big = xb.Shape(1, 8, 20, 20, 8, 8, 8)          # 64 taps
    with pytest.raises(xb.XnorError) as e:
        xb.xnor_conv2d_fp32_fwd(torch.zeros((1, 8, 20, 20), device="cuda"), torch.zeros((8, 8, 8, 8), device="cuda"), big,
                                algo=xb.ALGO_MFMA_SPLIT, workspace=ws)
    assert e.value.status == xb.E_UNSUPPORTED


def rel64(got, I, Wt, stride, pad):
    ref = torch.nn.functional.conv2d(torch.from_numpy(I).double(), torch.from_numpy(Wt).double(), stride=stride, padding=pad).numpy()
    return np.sqrt(((got - ref) ** 2).mean() / (ref ** 2).mean()), ((got - ref) / np.abs(ref)).mean()


@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("shape", [(2, 9, 30, 33, 24, 3), (2, 8, 30, 33, 24, 5), (4, 96, 14, 14, 40, 3), (1, 512, 14, 14, 64, 3), (2, 300, 9, 9, 64, 1),
                                   (2, 8, 30, 33, 24, 7), (2, 130, 12, 13, 40, 7), (1, 400, 14, 14, 32, 7)], ids=lambda s: "x".join(map(str, s)))
def test_split_is_no_less_exact_than_what_it_replaces(xb, shape, positive):
    """Against 64-bit sums, beside the kernel that runs without a workspace, on the same data.  The split form
    rounds an output's sum once per 32 terms (16 with one tap), the fp32 matrix instruction once per two: sqrt(2 / 32) = 0.25
    (0.35) of its error where roundings are independent, 0.16 to 0.57 measured; the form with short chains 0.3 to 0.5 of
    one thread per output.  Six products in the output's own chain are at 0.9 to 1.4, short chains without
    the rounding carried over at 7, a drift in the instruction's rounding left in at 1.0 to 1.6."""
    N, C, H, W, F, k = shape
    print(f"case conv_fp32 split exactness shape={shape} positive={positive}", flush=True)
    rng = np.random.default_rng(zlib.crc32(str(shape).encode()))
    I, Wt = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((F, C, k, k)).astype(np.float32)
    if positive:
        I, Wt = np.maximum(I, 0), np.abs(Wt)
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, k // 2, k // 2)
    replaced = xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, workspace=None).cpu().numpy().astype(np.float64)
    now, before = rel64(split(xb, dev(I), dev(Wt), s), I, Wt, 1, k // 2)[0], rel64(replaced, I, Wt, 1, k // 2)[0]
    assert now <= 0.75 * before, (now, before)


def test_split_products_of_equal_operands(xb):
    """Squares of values whose middle and last term have one sign and are both large: mid * lo and lo * mid are
    then together 2^-24 to 2^-25 of the product, and a split without them is that much low in every term.
    Channel sums of 64 such squares each; the roundings of the sums are of either sign and cancel in the
    mean over the values (3e-8 / sqrt(64) = 4e-9)."""
    print("case conv_fp32 split equal operands", flush=True)
    def bf16(x):
        return torch.from_numpy(x.astype(np.float32)).bfloat16().float().numpy().astype(np.float64)
    v = np.random.default_rng(2).uniform(1, 2, 20000).astype(np.float32).astype(np.float64)
    mid = bf16(v - bf16(v))
    lo = v - bf16(v) - mid
    v, mid, lo = (t[2 * mid * lo / v ** 2 >= 2.0 ** -25][:64] for t in (v, mid, lo))
    left_out = (2 * mid * lo / v ** 2).mean()
    assert v.size == 64 and left_out > 3e-8
    I = np.broadcast_to(v.astype(np.float32)[None, None, None, :], (1, 80, 1, 64)).copy()
    Wt = np.broadcast_to(v.astype(np.float32)[:, None, None, None], (64, 80, 1, 1)).copy()
    got = split(xb, dev(I), dev(Wt), xb.Shape(1, 80, 1, 64, 64, 1, 1))[0, :, 0, :].diagonal()
    bias = (got / (80 * v ** 2) - 1).mean()
    assert abs(bias) <= 0.5 * left_out, (bias, left_out)


@pytest.mark.parametrize("shape", [(1, 37, 14, 13, 70, 3), (2, 16, 9, 40, 33, 5), (1, 50, 15, 14, 66, 7)], ids=lambda s: "x".join(map(str, s)))
def test_split_weights_and_inputs_that_three_terms_do_not_hold(xb, shape):
    """Infinite, NaN, huge and tiny weights (and zeros beside them) in some filters, tiny values and regions of
    zeros in the input: what one thread per output gives, an infinite weight over padding adding nothing."""
    N, C, H, W, F, k = shape
    print(f"case conv_fp32 split weights shape={shape}", flush=True)
    rng = np.random.default_rng(11)
    I = np.maximum(rng.standard_normal((N, C, H, W)), 0).astype(np.float32)
    I[:, :, :k + 2, :k + 2] = 0
    I[:, C - 1, H - 2:, :] = 1e-40
    Wt = rng.standard_normal((F, C, k, k)).astype(np.float32)
    Wt[1, C - 1, 0, 0], Wt[2, 0, k - 1, 0], Wt[3, 1, 1, 1], Wt[33 % F, 2, 0, 0] = np.inf, -np.inf, np.nan, 3.402e38
    Wt[4], Wt[5], Wt[6, :, 1:], Wt[F - 1] = 0, Wt[5] * 1e-36, 0, Wt[F - 1] * 1e-42
    Wt[7, 0, 0, 0], Wt[8, 1, 0, 0] = 1e-44, 1e-34
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, k // 2, k // 2)
    ref = xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, algo=xb.ALGO_DIRECT).cpu().numpy().astype(np.float64)
    got = split(xb, dev(I), dev(Wt), s)
    assert np.isnan(ref).any() and np.isinf(ref).any() and np.isfinite(ref[:, 1]).any()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    # (a finite output has no weight that is not finite inside the image: S of the others)
    S = torch.nn.functional.conv2d(torch.from_numpy(I).double(), torch.from_numpy(np.where(np.isfinite(Wt), np.abs(Wt), 0)).double(),
                                   padding=k // 2).numpy()
    fine = np.isfinite(ref)
    assert (np.abs(got[fine] - ref[fine]) <= 1e-5 * S[fine] + 2 * C * k * k * 2.0 ** -149).all()


@pytest.mark.parametrize("what", ["one NaN", "all NaN", "overflow", "zeros and a tiny weight", "dead filters"])
@pytest.mark.parametrize("shape", [(16, 128, 28, 28, 128, 5), (16, 256, 28, 28, 256, 3), (4, 128, 28, 28, 128, 7)], ids=lambda s: "x".join(map(str, s)))
def test_split_costs_no_multiple_where_it_forms_outputs_again(xb, shape, what):
    """Outputs that the split cannot give are formed on the fp32 matrix instruction, a wave's at a time: 0.3 to 2.0
    times the whole call without a workspace.  One by one, as lanes' own sums, they took 3 to 80 times."""
    N, C, H, W, F, k = shape
    print(f"case conv_fp32 split cost shape={shape} {what}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    I, Wt = torch.randn((N, C, H, W), generator=g, device="cuda"), torch.randn((F, C, k, k), generator=g, device="cuda")
    if what == "one NaN":
        I[0, 5, 5, 5] = float("nan")
    elif what == "all NaN":
        I.fill_(float("nan"))
    elif what == "overflow":
        I, Wt = I * 1e25, Wt * 1e25
    elif what == "dead filters":
        Wt[::13] *= 1e-36
    else:
        I, Wt[::13, 0, 0, 0] = I.clamp(min=0), 1e-38
        I[:, :, :H // 2] = 0
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, k // 2, k // 2)
    out = torch.empty((N, F, H, W), device="cuda")
    best = {}
    for workspace in (None, "auto"):
        for _ in range(4):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            xb.xnor_conv2d_fp32_fwd(I, Wt, s, out, workspace=workspace)
            end.record()
            end.synchronize()
            best[workspace] = min(best.get(workspace, 1e9), start.elapsed_time(end))
    assert best["auto"] <= 2.8 * best[None], best


def test_split_by_name_with_the_default_workspace(xb):
    """ALGO_MFMA_SPLIT where ALGO_AUTO would not take it: the size can be asked for, and "auto" allocates it."""
    shape = (1, 3, 20, 21, 5, 3, 3, 1, 1, 1, 1)
    _, I, Wt = random_layer(np.random.default_rng(9), "t", *shape)
    s = xb.Shape(*shape)
    assert xb.xnor_conv2d_fp32_workspace_bytes(s) == 0
    nbytes = xb.xnor_conv2d_fp32_workspace_bytes(s, xb.ALGO_MFMA_SPLIT)
    assert nbytes > 0 and xb.xnor_conv2d_fp32_workspace_bytes(s, xb.ALGO_MFMA) == 0
    ws = torch.empty((nbytes,), dtype=torch.uint8, device="cuda")
    a = xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, algo=xb.ALGO_MFMA_SPLIT)
    b = xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, algo=xb.ALGO_MFMA_SPLIT, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and np.array_equal(a.cpu().numpy().astype(np.float64), split(xb, dev(I), dev(Wt), s))
    with pytest.raises(xb.XnorError) as e:
        xb.xnor_conv2d_fp32_fwd(dev(I), dev(Wt), s, algo=xb.ALGO_MFMA_SPLIT, workspace=None)
    assert e.value.status == xb.E_WORKSPACE
    big = xb.Shape(1, 8, 20, 20, 8, 8, 8)          # 64 taps
    with pytest.raises(xb.XnorError) as e:
        xb.xnor_conv2d_fp32_fwd(torch.zeros((1, 8, 20, 20), device="cuda"), torch.zeros((8, 8, 8, 8), device="cuda"), big,
                                algo=xb.ALGO_MFMA_SPLIT)
    assert e.value.status == xb.E_UNSUPPORTED


def test_auto_without_memory_for_the_workspace(xb, monkeypatch):
    """The default call works on a card that has no room for the split filters: the kernel that needs none."""
    s = xb.Shape(2, 64, 20, 20, 72, 3, 3, 1, 1, 1, 1)
    _, I, Wt = random_layer(np.random.default_rng(10), "t", 2, 64, 20, 20, 72, 3, 3, 1, 1, 1, 1)
    I, Wt, out = dev(I), dev(Wt), torch.empty((2, 72, 20, 20), device="cuda")
    assert xb.xnor_conv2d_fp32_workspace_bytes(s) > 0
    plain = xb.xnor_conv2d_fp32_fwd(I, Wt, s, workspace=None)

    def no_memory(*args, **kwargs):
        raise torch.OutOfMemoryError("no memory")
    monkeypatch.setattr(torch.Tensor, "new_empty", no_memory)
    xb.xnor_conv2d_fp32_fwd(I, Wt, s, out)
    with pytest.raises(torch.OutOfMemoryError):
        xb.xnor_conv2d_fp32_fwd(I, Wt, s, out, algo=xb.ALGO_MFMA_SPLIT)
    torch.cuda.synchronize()
    assert torch.equal(out, plain)


@pytest.mark.parametrize("shape", [(3, 17, 9, 11, 33, 1), (3, 48, 13, 12, 70, 3), (2, 33, 14, 15, 130, 5), (3, 16, 8, 9, 64, 2)], ids=lambda s: "x".join(map(str, s)))
def test_split_images_channels_and_filters_of_very_different_sizes(xb, shape):
    """The powers of two that an image and a filter chunk are multiplied by: images of 1e-25 .. 1e15, a channel and a
    corner far below or above the rest, filters and chunks of filters likewise, zeros.  Against 64-bit sums: an output's
    sum is rounded once per chain of two taps and 16 channels, a chain's about six times (each by at most 2^-23 of S, the
    sum of |I * Wt|), and the smallest products lose at most 2^-24 together: (chains + 8) * 2^-23 * S; an output
    formed again by the plain sum is rounded once per two terms."""
    N, C, H, W, F, k = shape
    print(f"case conv_fp32 split sizes shape={shape}", flush=True)
    rng = np.random.default_rng(zlib.crc32(("sizes" + str(shape)).encode()))
    I, Wt = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((F, C, k, k)).astype(np.float32)
    for n, size in zip(range(N), (1e-25, 1e15, 1.0)):
        I[n] *= np.float32(size)
    I[:, C // 2] *= np.float32(1e-9)
    I[N - 1, 0, :2, :2] *= np.float32(1e12)
    I[0, :, H // 2] = 0
    Wt[1] *= np.float32(1e-7)
    Wt[2, : C // 2] *= np.float32(1e-12)
    Wt[F // 2] = 0
    Wt[:, C - 1] *= np.float32(1e6)
    Wt[min(F - 1, 32):, : min(C, 16)] *= np.float32(1e-4)
    s = xb.Shape(N, C, H, W, F, k, k, 1, 1, k // 2, k // 2)
    got = split(xb, dev(I), dev(Wt), s)
    d = [torch.from_numpy(a).double() for a in (I, Wt)]
    ref = torch.nn.functional.conv2d(*d, padding=k // 2).numpy()
    S = torch.nn.functional.conv2d(d[0].abs(), d[1].abs(), padding=k // 2).numpy()
    chains = (k * k + 1) // 2 * -(-C // 16)
    bar = max(chains + 8, C * k * k / 2 + 8) * 2.0 ** -23 * S
    assert (np.abs(got - ref) <= bar + 2.0 ** -149).all()
    assert np.sqrt(((got - ref) ** 2).sum()) <= 3e-7 * np.sqrt((S ** 2).sum())


def sums64(I, Wt, pad):
    d = [torch.from_numpy(a).double() for a in (I, Wt)]
    return [torch.nn.functional.conv2d(*x, padding=pad).numpy() for x in (d, [v.abs() for v in d])]


@pytest.mark.parametrize("k", [1, 2, 3, 5])
def test_split_filter_far_below_the_others(xb, k):
    """A filter 2^-40 of its neighbours is summed from the same products as at their size: its outputs are the same bits
    but for the exponent (its tile holds another such filter in both runs, so that both take the same products)."""
    print(f"case conv_fp32 split far below k={k}", flush=True)
    rng = np.random.default_rng(21)
    I, Wt = rng.standard_normal((2, 40, 11, 12)).astype(np.float32), rng.standard_normal((70, 40, k, k)).astype(np.float32)
    Wt[[1, 40, 66]] *= np.float32(2.0 ** -45)
    s = xb.Shape(2, 40, 11, 12, 70, k, k, 1, 1, k // 2, k // 2)
    a = split(xb, dev(I), dev(Wt), s)
    Wt[[5, 69]] *= np.float32(2.0 ** -40)
    b = split(xb, dev(I), dev(Wt), s)
    assert np.array_equal(b[:, [5, 69]] * 2.0 ** 40, a[:, [5, 69]])
    ref, S = sums64(I, Wt, k // 2)
    chains = (k * k + 1) // 2 * 3
    assert (np.abs(b - ref) <= (chains + 8) * 2.0 ** -23 * S).all()


@pytest.mark.parametrize("what", ["first_zero", "first_tiny", "first_large", "tiny_later", "large_later", "largest_later", "half_zero", "top_meets_zero"])
@pytest.mark.parametrize("shape", [(2, 40, 9, 11, 33, 1), (2, 70, 13, 12, 130, 2), (1, 100, 14, 15, 70, 3), (2, 33, 8, 9, 64, 5)], ids=lambda s: "x".join(map(str, s)))
def test_split_inputs_far_from_the_first_chunk(xb, shape, what):
    """The workgroup's power of two comes from its first 16 channels: nothing, values far below and far above the others
    there, and values outside what f16 holds from some later channel on.  Bar: a sum is rounded once per chain of two taps and
    16 channels, a chain's about six times, each by at most 2^-23 of S = sum |I * Wt|; the plain sum once per two terms."""
    N, C, H, W, F, k = shape
    print(f"case conv_fp32 split first chunk shape={shape} {what}", flush=True)
    rng = np.random.default_rng(zlib.crc32((what + str(shape)).encode()))
    I, Wt = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((F, C, k, k)).astype(np.float32)
    if what == "first_zero":
        I[:, :16] = 0
    if what == "first_tiny":
        I[:, :16] *= np.float32(1e-37)
    if what == "first_large":
        I[:, :16] *= np.float32(1e33)
        I[0, :16, : H // 2] = 0
    if what == "tiny_later":
        I[:, C - 2, 2, 3] = 1e-20
    if what == "large_later":
        I[:, C - 2, 2, 3] = 1e9
    if what == "largest_later":
        I[:, :16] *= np.float32(1e-30)
        I[:, C - 2, 2, 3] = 1e36
    if what == "half_zero":
        I[:, :, H // 2:] = 0
        I[:, 0, 0, 0] = 1e-12
    if what == "top_meets_zero":        # a value of 2^126 that meets weights of 0, beside weights of 2^60: their product is no float
        I[:, 0] = 1e38
        Wt *= np.float32(2.0 ** 60)
        Wt[:, 0] = 0
    got = split(xb, dev(I), dev(Wt), xb.Shape(N, C, H, W, F, k, k, 1, 1, k // 2, k // 2))
    ref, S = sums64(I, Wt, k // 2)
    chains = (k * k + 1) // 2 * -(-C // 16)
    assert (np.abs(got - ref) <= max(chains + 8, C * k * k / 2 + 8 if what in ("first_large", "largest_later") else 0) * 2.0 ** -23 * S + 2.0 ** -149).all()
    assert np.sqrt(((got - ref) ** 2).sum()) <= 3e-7 * np.sqrt((S ** 2).sum())


def test_split_more_positions_than_three_granules(xb):
    """32 pixels over more than 384 staged positions (wide strides): the variant that fetches four granules ahead."""
    for shape in ((1, 64, 19, 202, 24, 3, 3, 4, 5, 3, 0), (3, 20, 67, 49, 200, 4, 4, 4, 5, 4, 4), (2, 8, 67, 174, 9, 5, 3, 4, 4, 2, 3)):
        print(f"case conv_fp32 split positions shape={shape}", flush=True)
        _, I, Wt = random_layer(np.random.default_rng(12), "t", *shape)
        O, S = oracle.conv_fp32(I, Wt, oracle.Shape(*shape), want_scale=True)
        got = split(xb, dev(I), dev(Wt), xb.Shape(*shape))
        assert (np.abs(got - O) <= 1e-5 * S).all()
