"""xnor_forward_image on several filters where tiles of output pixels are taken: edges of the tiles, of
the 64-column units they are staged in and of the filter groups, against the oracle (bars as in
tests/test_gpu_image.py)."""
import pytest
import torch

from test_gpu_image import run_case, xb  # noqa: F401  (xb: the fixture)

pytestmark = pytest.mark.gpu

#   N  C   H    W   F  k  pad (sh sw)
SHAPES = [
    (1, 2, 3, 3, 16, 3, 1),             # an image of one tile, nine pixels
    (1, 4, 1, 1, 17, 7, 3, 2, 2),       # one pixel, everything else padding
    (1, 3, 40, 256, 16, 3, 1),          # rows of exactly one tile
    (2, 3, 9, 257, 19, 3, 1),           # one pixel more: two tiles a row, the second ragged
    (1, 2, 5, 700, 33, 5, 2),           # three tiles a row
    (3, 3, 61, 62, 16, 3, 0),           # 60 columns: staged rows of 62
    (1, 3, 30, 64, 24, 7, 3),           # staged rows of 70: two 64-column units
    (2, 3, 33, 35, 65, 7, 6),           # padding nearly as wide as the window
    (1, 4, 29, 31, 40, 5, 8, 2, 3),     # windows that are all padding, unequal strides
    (1, 4, 50, 51, 300, 5, 2),          # more filters than a group holds
    (1, 3, 200, 190, 8, 5, 2),          # two pixels per lane
    (16, 3, 115, 117, 64, 7, 3, 2, 2),
    (1, 3, 900, 3000, 20, 7, 3, 9, 11), # strides so large that a tile has to shrink to fit the LDS
    (1, 4, 130, 128, 2, 7, 0, 4, 4),    # few filters, strided
    (4, 3, 79, 69, 49, 3, 1, 4, 4),     # few workgroups: tiles of what one batch of loads stages
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_tiles_vs_oracle(xb, shape):  # noqa: F811
    print(f"case image tiles shape={shape}", flush=True)
    run_case(xb, shape, "tiles")


def test_tiles_values_that_are_not_numbers(xb):  # noqa: F811
    """NaN counts as -1 and makes the outputs under it NaN, as in the one-filter kernel; all others stay."""
    s = xb.Shape(1, 3, 40, 40, 16, 3, 3, 1, 1, 1, 1)
    g = torch.Generator().manual_seed(3)
    I, Wt = torch.randn((1, 3, 40, 40), generator=g), torch.randn((16, 3, 3, 3), generator=g)
    Wpk, alpha, _ = xb.xnor_filter_prepare(Wt.cuda())
    out, dot = xb.xnor_forward_image(I.cuda(), Wpk, alpha, s, want_dot=True)
    I[0, 1, 20, 20] = float("nan")
    out2, dot2 = xb.xnor_forward_image(I.cuda(), Wpk, alpha, s, want_dot=True)
    I[0, 1, 20, 20] = -1.0
    _, dot3 = xb.xnor_forward_image(I.cuda(), Wpk, alpha, s, want_dot=True)
    torch.cuda.synchronize()
    under = torch.zeros((40, 40), dtype=torch.bool, device="cuda")
    under[19:22, 19:22] = True
    assert torch.equal(torch.isnan(out2), under.expand_as(out2))
    assert torch.equal(out[..., ~under], out2[..., ~under]) and torch.equal(dot2, dot3)


#   N  C   H    W   F  k  pad: one channel, one filter, rows of whole 16 bytes, half a million pixels and more
ROW4 = [
    (1, 1, 131072, 4, 1, 3, 1),         # one lane per row: both neighbours are the image's edge
    (1, 1, 2051, 256, 1, 3, 1),         # one wave per row, the last band short
    (3, 1, 700, 260, 1, 3, 1),          # a lane past the wave's 256 columns
    (2, 1, 261, 1020, 1, 5, 2),         # two columns from either side
    (150000, 1, 1, 4, 1, 5, 2),         # images lower than the window
    (1, 1, 1300, 508, 1, 5, 2),
]


@pytest.mark.parametrize("shape", ROW4, ids=lambda s: "x".join(map(str, s)))
def test_four_columns_per_lane_vs_oracle(xb, shape):  # noqa: F811
    print(f"case image row4 shape={shape}", flush=True)
    run_case(xb, shape, "row4")


def test_four_columns_per_lane_match_one_column(xb):  # noqa: F811
    """The same image at an address that is no multiple of 16 goes through the one-column kernel: bit for bit the same."""
    s = xb.Shape(1, 1, 800, 1024, 1, 3, 3, 1, 1, 1, 1)
    I = torch.randn((1, 1, 800, 1024), generator=torch.Generator().manual_seed(4)).cuda()
    Wpk, alpha, _ = xb.xnor_filter_prepare(torch.randn((1, 1, 3, 3), generator=torch.Generator().manual_seed(5)).cuda())
    shifted = torch.empty(800 * 1024 + 1, device="cuda")[1:].view(1, 1, 800, 1024)
    shifted.copy_(I)
    a, da = xb.xnor_forward_image(I, Wpk, alpha, s, want_dot=True)
    b, db = xb.xnor_forward_image(shifted, Wpk, alpha, s, want_dot=True)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(da, db)
