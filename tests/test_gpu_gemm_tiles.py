"""GPU: the tiles of the bf16 product (256 x 256, 128 x 128, 128 x 256 in the in-LDS recover form) at ragged edges, with one,
several and many K-slices, as a fully-connected layer and read through a convolution's window, against the same product in
64 bits.  Sums of n exact products in fp32 err by about sqrt(n) 2^-24 of the terms: 2e-6 in the 2-norm covers 50176 tokens."""
import pytest
import torch

import paper_2202_13808_amd as dropit

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def recovered(vals, idx, shape):
    flat = torch.zeros(torch.Size(shape).numel(), dtype=torch.float64, device=DEV)
    flat[idx.long()] = vals.double()
    return flat.reshape(shape)


def inputs(x_shape, dy_shape, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn(x_shape, generator=gen, device=DEV).relu_().bfloat16()
    return x, (torch.randn(dy_shape, generator=gen, device=DEV) * 0.02).bfloat16()


def check(got, want, what):
    err = ((got.double() - want).norm() / want.norm()).item()
    print("gemm tiles", what, "%.2e" % err, flush=True)
    assert err < 2e-6


@pytest.mark.parametrize("ntok,cin,cout", [
    (9589, 1381, 1928),       # the wide tile, ragged in all three dimensions, several slices
    (2041, 3069, 3064),       # the wide tile, one slice straight into dW
    (300, 200, 136),          # the small tile: just over one tile in both dimensions
    (129, 127, 128),          # ... exactly one row of tiles, a partial column, a partial token block
    (33, 2305, 1160),         # ... two token blocks in many tiles, one slice
    (20001, 264, 72),         # ... more than 16 slices
    (3150, 776, 3000),        # ... cut so that two workgroups share every compute unit
    (8312, 1208, 360),
])
def test_fully_connected(ntok, cin, cout):
    x, dy = inputs((ntok, cin), (ntok, cout), ntok)
    vals, idx = dropit.compress(x, 0.8)
    assert dropit.weight_grad_path(x.shape, x.dtype, vals.numel(), cout) == "fc_mfma"
    want = dy.double().t() @ recovered(vals, idx, x.shape)
    dense = dropit.weight_grad(vals, idx, x.shape, dy, cout)
    check(dense, want, (ntok, cin, cout))
    if cout > 128:                                 # the in-LDS form: the same slices in tiles of its own
        dropit.set_fc_recover(1)
        try:
            fused = dropit.weight_grad(vals, idx, x.shape, dy, cout)
        finally:
            dropit.set_fc_recover(0)
        assert torch.equal(dense, fused)


@pytest.mark.parametrize("layout,n,c,h,w,j,stride", [
    ("nhwc", 3, 24, 17, 15, 40, 1),        # one partial tile of rows, ragged taps
    ("nhwc", 5, 136, 19, 23, 136, 2),
    ("nhwc", 64, 512, 7, 7, 512, 1),       # slices raised until two workgroups share every compute unit
    ("nchw", 64, 512, 7, 7, 512, 1),       # ... and channel-major dW
    ("nchw", 3, 136, 9, 11, 136, 1),       # small tile, channel-major, few slices
    ("nchw", 64, 256, 14, 14, 264, 1),
])
def test_through_the_window(layout, n, c, h, w, j, stride):
    oh, ow = (h - 1) // stride + 1, (w - 1) // stride + 1
    conv = (3, 3, stride, stride, 1, 1, 1, 1)
    xs, ys = ((n, h, w, c), (n, oh, ow, j)) if layout == "nhwc" else ((n, c, h, w), (n, j, oh, ow))
    x, dy = inputs(xs, ys, n + c)
    vals, idx = dropit.compress(x, 0.8)
    got = dropit.weight_grad(vals, idx, xs, dy, j, conv=conv, layout=layout)
    xr, yr = recovered(vals, idx, xs), dy.double()
    if layout == "nhwc":
        xr, yr = xr.permute(0, 3, 1, 2), yr.permute(0, 3, 1, 2)
    cols = torch.nn.functional.unfold(xr.contiguous(), 3, padding=1, stride=stride)           # [n, c * 9, positions]
    want = (yr.reshape(n, j, -1).transpose(0, 1).reshape(j, -1) @ cols.transpose(1, 2).reshape(-1, c * 9)).reshape(j, c, 3, 3)
    if layout == "nhwc":
        want = want.permute(0, 2, 3, 1)
    check(got, want.contiguous(), (layout, n, c, h, w, j, stride))


@pytest.mark.parametrize("ntok,cin,cout", [
    (121, 1800, 80), (288, 136, 264), (289, 500, 136),      # few blocks: one slice straight into dW, in small tiles
    (480, 629, 1440),                                       # ... more of them in more tiles
    (1900, 2224, 1304),                                     # rows of more than sixteen small tiles
])
def test_one_slice_and_long_rows(ntok, cin, cout):
    test_fully_connected(ntok, cin, cout)


@pytest.mark.parametrize("n,c,h,w,j", [(1, 128, 14, 14, 256), (2, 256, 9, 9, 136), (1, 512, 4, 5, 1032)])
def test_channel_major_results_of_few_blocks(n, c, h, w, j):
    """The slice sum runs for these whatever the slices: it writes dW [J][C][taps]."""
    test_through_the_window("nchw", n, c, h, w, j, 1)
