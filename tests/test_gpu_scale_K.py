"""xnor_scale_K of small inputs, in one launch: at the edges of its bands, against the oracle, and K bit for bit what
xnor_box_filter_K makes of the same A."""
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
