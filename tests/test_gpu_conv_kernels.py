"""Each of the three matrix-core convolution kernels by name, over the shape lists of the parity, chain and random
tests, whichever of them the dispatch takes for a shape: with K, with A, with filters expanded beforehand and in
the chained form, against the oracle and against each other (one expression on the same exact dot: the same bits).

Layers of little work run on the small workgroups, so lists of layers that the oracle finishes in seconds reach
the persistent workgroups and the bands by name only; test_dispatch says which kernel a shape's default is."""
import zlib

import numpy as np
import pytest
import torch

import oracle
from paper_2007_14178_amd.workloads import LAYERS, random_layer
from test_gpu_chain import SHAPES as CHAIN_SHAPES
from test_gpu_conv_tile import SHAPES as TILE_SHAPES
from test_gpu_parity import SHAPES as PARITY_SHAPES
from test_gpu_random_shapes import cases

pytestmark = pytest.mark.gpu
RTOL = 1e-5
KERNELS = ["tile", "persistent", "bands"]


@pytest.fixture(scope="module")
def xb():
    from paper_2007_14178_amd import binding
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def algo_id(xb, kernel):
    return {"tile": xb.ALGO_MFMA_TILE, "persistent": xb.ALGO_MFMA_PERSISTENT, "bands": xb.ALGO_MFMA_BANDS}[kernel]


_REF: dict = {}


def reference(shape):
    if shape not in _REF:
        _REF.clear()
        rng = np.random.default_rng(zlib.crc32(("kernels" + str(shape)).encode()))
        _, I, Wt = random_layer(rng, "k", *shape)
        d, K, a, O = oracle.forward(I, Wt, oracle.Shape(*shape))
        floor = (0.5 * np.abs(d.astype(np.float64)) * (a.astype(np.float64)[None, :, None, None] + 1.0) + 1.0) * 2.0 ** -149
        _REF[shape] = I, Wt, d, O.astype(np.float64), np.maximum(RTOL * np.abs(O.astype(np.float64)), floor)
    return _REF[shape]


def misaligned(t, words):
    buf = torch.empty((t.numel() + 4,), dtype=t.dtype, device="cuda")
    v = buf[words:words + t.numel()].view(t.shape)
    v.copy_(t)
    return v


def check(xb, shape, kernel, words=0):
    s, algo = xb.Shape(*shape), algo_id(xb, kernel)
    nbytes = xb.xnor_conv2d_algo_workspace_bytes(s, algo)
    if nbytes == 0:
        pytest.skip(f"{kernel} does not take this shape")
    I, Wt, d_ref, O_ref, bar = reference(shape)
    Ipk, K, A = xb.xnor_input_prepare(dev(I), s)
    if words:
        Ipk = misaligned(Ipk, words)
    Wpk, alpha, _ = xb.xnor_filter_prepare(dev(Wt))
    out, dot = xb.xnor_conv2d_fwd(Ipk, Wpk, K, alpha, s, want_dot=True, algo=algo)
    ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda")
    xb.xnor_filter_expand(Wpk, s, ws, algo=algo)
    alone, _ = xb.xnor_conv2d_fwd_expanded(Ipk, ws, K, alpha, s, algo=algo)
    outA, dotA = xb.xnor_conv2d_fwd_expanded(Ipk, ws, None, alpha, s, want_dot=True, A=A, algo=algo)
    Opk, A_next = xb.xnor_conv2d_fwd_chain(Ipk, Wpk, K, alpha, s, algo=algo)
    cws = torch.full((xb.xnor_conv2d_algo_workspace_bytes(s, algo, chained=True),), 0x5A, dtype=torch.uint8, device="cuda")
    xb.xnor_filter_expand(Wpk, s, cws, algo=algo)
    OpkA, A_nextA = xb.xnor_conv2d_fwd_chain(Ipk, None, None, alpha, s, workspace=cws, A=A, algo=algo)
    torch.cuda.synchronize()
    assert np.array_equal(dot.cpu().numpy(), d_ref) and torch.equal(dotA, dot)
    got = out.cpu().numpy()
    assert (np.abs(got.astype(np.float64) - O_ref) <= bar).all()
    assert torch.equal(alone, out) and torch.equal(outA, out)
    direct, _ = xb.xnor_conv2d_fwd(Ipk, Wpk, K, alpha, s, algo=xb.ALGO_DIRECT)
    assert torch.equal(direct, out)
    assert np.array_equal(Opk.cpu().numpy().view(np.uint32), oracle.pack(got)) and torch.equal(OpkA, Opk)
    mean = np.abs(got.astype(np.float64)).mean(axis=1)
    assert (np.abs(A_next.cpu().numpy() - mean) <= np.maximum(RTOL * mean, 2.0 ** -149)).all() and torch.equal(A_next, A_nextA)


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("shape", sorted(set(PARITY_SHAPES + CHAIN_SHAPES + TILE_SHAPES)), ids=lambda s: "x".join(map(str, s)))
def test_listed_shapes(xb, shape, kernel):
    print(f"case kernel={kernel} shape={shape}", flush=True)
    check(xb, shape, kernel)


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("shape", cases()[::3], ids=lambda s: "x".join(map(str, s)))
def test_random_shapes(xb, shape, kernel):
    print(f"case kernel={kernel} random shape={shape}", flush=True)
    check(xb, shape, kernel)


@pytest.mark.parametrize("words", [1, 2, 3])
@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("shape", [(2, 128, 28, 28, 64, 3, 3, 1, 1, 1, 1), (5, 256, 14, 14, 130, 3, 3, 1, 1, 1, 1), (1, 512, 28, 28, 96, 3, 3, 1, 1, 1, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_input_that_is_not_16_byte_aligned(xb, shape, kernel, words):
    print(f"case kernel={kernel} misaligned by {words} words shape={shape}", flush=True)
    check(xb, shape, kernel, words)


@pytest.mark.parametrize("kernel", KERNELS)
def test_infinite_K(xb, kernel):
    """Chained, a partly filled filter tile: infinity (and signs) where K is infinite, on every kernel."""
    shape = (2, 33, 12, 11, 75, 3, 3, 1, 1, 1, 1)
    print(f"case kernel={kernel} infinite K", flush=True)
    _, I, Wt = random_layer(np.random.default_rng(75), "t", *shape)
    I[0, 7, 5, 5] = np.inf
    s, algo = xb.Shape(*shape), algo_id(xb, kernel)
    Ipk, K, _ = xb.xnor_input_prepare(dev(I), s)
    Wpk, alpha, _ = xb.xnor_filter_prepare(dev(Wt))
    Opk, A_next = xb.xnor_conv2d_fwd_chain(Ipk, Wpk, K, alpha, s, algo=algo)
    with np.errstate(all="ignore"):
        _, _, _, O = oracle.forward(I, Wt, oracle.Shape(*shape))
    assert np.array_equal(Opk.cpu().numpy().view(np.uint32), oracle.pack(O))
    infinite = np.zeros((2, 12, 11), dtype=bool)
    infinite[0, 4:7, 4:7] = True
    A_next = A_next.cpu().numpy()
    assert np.isinf(A_next[infinite]).all() and np.isfinite(A_next[~infinite]).all()


def test_dispatch(xb):
    """Which kernel the default is: the small workgroups for the lists above, the other two beyond 18.5 k cycles of
    matrix work per SIMD."""
    def kernel(*shape):
        return xb.xnor_conv2d_mfma_kernel(xb.Shape(*shape))
    for shape in TILE_SHAPES:
        assert kernel(*shape) == xb.ALGO_MFMA_TILE, shape
    assert sum(kernel(*c) == xb.ALGO_MFMA_TILE for c in cases() if xb.xnor_conv2d_workspace_bytes(xb.Shape(*c))) >= 100
    c5 = LAYERS["c5"]
    full = (c5.N, c5.C, c5.H, c5.W, c5.F, c5.kh, c5.kw, c5.sh, c5.sw, c5.ph, c5.pw)
    assert kernel(*full) == xb.ALGO_MFMA_PERSISTENT
    assert kernel(128, 96, 27, 27, 256, 5, 5, 1, 1, 2, 2) != xb.ALGO_MFMA_TILE
    s = xb.Shape(*full)
    assert xb.xnor_conv2d_workspace_bytes(s) >= xb.xnor_conv2d_algo_workspace_bytes(s, xb.ALGO_MFMA_PERSISTENT) > 0
    for algo in (xb.ALGO_AUTO, xb.ALGO_DIRECT, xb.ALGO_TILED, xb.ALGO_MFMA_SPLIT):
        assert xb.xnor_conv2d_algo_workspace_bytes(s, algo) == 0
