"""xnor_scale_K of small inputs, in one launch: at the edges of its bands, against the oracle, and K bit for bit what
xnor_box_filter_K makes of the same A."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2007_14178_amd.workloads import random_layer

pytestmark = pytest.mark.gpu

#        N   C   H   W   F  kh kw sh sw ph pw
SHAPES = [
    (1, 1, 1, 1, 1, 1, 1, 1, 1, 0, 0),
    (1, 64, 32, 32, 64, 3, 3, 1, 1, 1, 1),       # a band of one row
    (6, 100, 37, 53, 75, 3, 3, 1, 1, 1, 1),      # two launches: more than 2^20 values
    (5, 100, 37, 53, 75, 3, 3, 1, 1, 1, 1),      # one: odd rows and channels
    (300, 7, 5, 9, 3, 3, 3, 1, 1, 1, 1),         # more images than blocks are asked for: a band of all rows
    (2, 33, 61, 7, 3, 5, 3, 1, 1, 2, 1),
    (1, 20, 40, 11, 3, 3, 3, 5, 2, 0, 1),        # rows that no window touches
    (1, 20, 41, 11, 3, 3, 3, 5, 2, 0, 1),
    (2, 17, 6, 5, 3, 3, 3, 1, 1, 7, 7),          # windows that are all padding
    (1, 8, 9, 200, 3, 9, 9, 1, 1, 4, 4),         # bands that read every row: two launches
    (1, 256, 20, 20, 3, 3, 3, 2, 2, 1, 1),       # sixteen slices
    (1, 3, 500, 600, 3, 7, 7, 1, 1, 3, 3),
    (1, 9, 3, 9000, 3, 3, 3, 1, 1, 1, 1),        # rows that LDS does not hold
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_scale_K_of_small_inputs(shape):
    from paper_2007_14178_amd import binding as xb
    print(f"case scale_K shape={shape}", flush=True)
    _, I, _ = random_layer(np.random.default_rng(sum(shape)), "t", *shape)
    s, so = xb.Shape(*shape), oracle.Shape(*shape)
    dI = torch.from_numpy(I).cuda()
    A, K = torch.full((s.N, s.H, s.W), float("nan"), device="cuda"), torch.full((s.N, *xb.xnor_out_dim(s)), float("nan"), device="cuda")
    xb.xnor_scale_K(dI, s, A, K)
    torch.cuda.synchronize()
    assert torch.equal(K, xb.xnor_box_filter_K(A, s))
    for got, ref in ((A, oracle.channel_mean_abs(I)), (K, oracle.scale_K(I, so))):
        ref = np.asarray(ref, dtype=np.float64)
        assert (np.abs(got.cpu().numpy() - ref) <= np.maximum(1e-5 * np.abs(ref), 2.0 ** -149)).all()


#        N   C   H   W   F  kh kw sh sw ph pw, launches
ROUTES = [
    ((1, 64, 32, 32, 64, 3, 3, 1, 1, 1, 1), 1),
    ((64, 4, 9, 7, 3, 3, 3, 1, 1, 1, 1), 1),       # bands of three rows
    ((1, 16, 30, 85, 3, 3, 3, 1, 1, 1, 1), 1),     # two slices of eight groups, 255 pixels
    ((1, 7, 90, 682, 3, 3, 3, 1, 1, 1, 1), 1),     # all pixels of sixteen groups but two
    ((1, 7, 90, 683, 3, 3, 3, 1, 1, 1, 1), 2),     # more pixels than threads take
    ((1, 768, 9, 21, 3, 3, 3, 1, 1, 1, 1), 1),     # one pixel, 48 channels each
    ((1, 784, 9, 21, 3, 3, 3, 1, 1, 1, 1), 1),     # 49, few values in all
    ((16, 1023, 8, 8, 3, 3, 3, 1, 1, 1, 1), 2),    # 64, many
    ((1, 2045, 20, 20, 3, 3, 3, 1, 1, 1, 1), 1),
    ((1, 1, 1000, 1000, 3, 3, 3, 1, 1, 1, 1), 1),  # one channel: three passes
    ((1, 1, 100, 2500, 3, 3, 3, 1, 1, 1, 1), 2),   # on fewer units
    ((1, 256, 9, 42, 3, 3, 3, 1, 1, 1, 1), 1),     # two pixels, 16 channels each
    ((1, 272, 9, 42, 3, 3, 3, 1, 1, 1, 1), 2),     # 17
    ((300, 7, 5, 9, 3, 3, 3, 1, 1, 1, 1), 2),      # more bands than units
    ((1, 512, 1, 2000, 3, 1, 1, 1, 1, 0, 0), 2),   # one output row: all the reads in one workgroup
    ((1, 116, 3, 3000, 3, 3, 3, 1, 1, 1, 1), 2),   # three
    ((1, 64, 7, 1500, 3, 7, 7, 1, 1, 0, 0), 2),
    ((1, 1024, 28, 28, 3, 3, 3, 1, 1, 1, 1), 2),
]


@pytest.mark.parametrize("shape, launches", ROUTES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_scale_K_takes_one_launch_where_no_workgroup_has_much_to_read(shape, launches):
    """Launches counted as nodes of a captured graph, whose replays give the eager call's values on new inputs."""
    from paper_2007_14178_amd import binding as xb
    print(f"case scale_K route shape={shape}", flush=True)
    s, so = xb.Shape(*shape), oracle.Shape(*shape)
    rng = np.random.default_rng(sum(shape))
    I = torch.zeros((s.N, s.C, s.H, s.W), device="cuda")
    A, K = torch.empty((s.N, s.H, s.W), device="cuda"), torch.empty((s.N, *xb.xnor_out_dim(s)), device="cuda")
    xb.xnor_scale_K(I, s, A, K)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        xb.xnor_scale_K(I, s, A, K)
    nodes = ctypes.c_size_t()
    assert xb.lib.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert nodes.value == launches
    graph.instantiate()
    for _ in range(2):
        x = random_layer(rng, "t", *shape)[1]
        I.copy_(torch.from_numpy(x))
        A.fill_(float("nan"))
        K.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(K, xb.xnor_box_filter_K(A, s))
        for got, ref in ((A, oracle.channel_mean_abs(x)), (K, oracle.scale_K(x, so))):
            ref = np.asarray(ref, dtype=np.float64)
            assert (np.abs(got.cpu().numpy() - ref) <= np.maximum(1e-5 * np.abs(ref), 2.0 ** -149)).all()
