"""GPU: the exact fp32 product (fp32 tensors, and bf16 shapes the bf16 matrix-core paths do not take) at the edges of
its tiles, token steps and K-slices, element by element against the fp64 oracle.

Bound per element: an fp32 sum of n products, in any order and with any grouping, is within n * 2^-24 of the exact
sum relative to the sum of the terms' magnitudes (n * u / (1 - n * u), u = 2^-24).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import activation, f32_to_bf16_bits, gradient
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


def check(x, dy, gamma, c_out, dense_dw, terms, conv=None, layout="nchw"):
    xd, dyd = to_device(x), to_device(dy)
    vals, idx = dropit.compress(xd, gamma)
    assert dropit.weight_grad_path(x.shape, xd.dtype, vals.numel(), c_out, conv, layout=layout) == "fma"
    dW = dropit.weight_grad(vals, idx, x.shape, dyd, c_out, conv=conv, layout=layout)
    torch.cuda.synchronize()
    k = oracle.keep_count(x.size, gamma)
    xh = oracle.densify(*oracle.compress(x, k), x.shape)
    ref, size = dense_dw(xh, oracle.widen(dy)), dense_dw(np.abs(xh), np.abs(oracle.widen(dy)))
    nu = (terms + 256) * 2.0 ** -24                     # the terms of a sum, and the K-slices that meet in it
    excess = np.abs(to_host(dW).astype(np.float64) - ref) - nu / (1 - nu) * size
    assert excess.max() <= 0.0, excess.max()


@pytest.mark.parametrize("dtype,ntok,cin,cout", [
    ("f32", 31, 1000, 129), ("f32", 32, 516, 128), ("f32", 33, 516, 132), ("f32", 4001, 64, 64), ("f32", 2048, 61, 67),
    ("f32", 20000, 12, 4), ("f32", 700, 130, 2), ("bf16", 1025, 130, 129), ("bf16", 3000, 63, 9)])
def test_fc_tile_edges(dtype, ntok, cin, cout):
    print("exact fc", dtype, ntok, cin, cout, flush=True)
    x, dy = activation((ntok, cin), "normal", 11 + ntok, dtype), gradient((ntok, cout), 0.02, 12 + ntok, dtype)
    check(x, dy, 0.7, cout, oracle.dw_fc, ntok)


@pytest.mark.parametrize("gamma", [0.0, 0.9])
@pytest.mark.parametrize("dtype,ntok,cin,cout", [
    ("f32", 65, 1009, 3), ("f32", 257, 1021, 2), ("f32", 300, 3500, 5), ("bf16", 47, 372, 5), ("bf16", 33, 32001, 9),
    ("f32", 8200, 257, 3), ("f32", 390, 72, 96), ("f32", 16384, 129, 1)])
def test_small_recover_tiles_and_slices(dtype, ntok, cin, cout, gamma):
    """Recover tiles of 1024 elements up to the largest, with the tensor's end inside one; slices of one step and of two."""
    print("exact small tiles", dtype, ntok, cin, cout, gamma, flush=True)
    x, dy = activation((ntok, cin), "normal", 13 + ntok, dtype), gradient((ntok, cout), 0.02, 14 + ntok, dtype)
    check(x, dy, gamma, cout, oracle.dw_fc, ntok)


@pytest.mark.parametrize("dtype,layout,shape,J,geom", [
    ("f32", "nchw", (3, 7, 9, 11), 5, (3, 3, 1, 1, 1, 1, 1, 1)), ("f32", "nchw", (2, 64, 16, 16), 64, (3, 3, 1, 1, 1, 1, 1, 1)),
    ("f32", "nchw", (1, 15, 33, 31), 130, (3, 2, 2, 1, 0, 1, 1, 2)), ("f32", "nhwc", (3, 15, 17, 33), 66, (3, 3, 2, 2, 1, 1, 1, 1)),
    ("f32", "nhwc", (2, 12, 12, 20), 64, (1, 1, 2, 2, 0, 0, 1, 1)), ("bf16", "nchw", (2, 9, 13, 10), 12, (5, 3, 1, 2, 2, 1, 1, 1)),
    ("bf16", "nhwc", (2, 13, 10, 24), 7, (3, 3, 1, 1, 2, 0, 2, 1))])
def test_conv_geometries(dtype, layout, shape, J, geom):
    print("exact conv", dtype, layout, shape, J, geom, flush=True)
    kh, kw, sh, sw, ph, pw, dh, dw = geom
    H, W = (shape[1], shape[2]) if layout == "nhwc" else (shape[2], shape[3])
    OH, OW = (H + 2 * ph - dh * (kh - 1) - 1) // sh + 1, (W + 2 * pw - dw * (kw - 1) - 1) // sw + 1
    x = activation(shape, "relu", 21 + H, dtype)
    dy = gradient((shape[0], OH, OW, J) if layout == "nhwc" else (shape[0], J, OH, OW), 0.02, 22 + W, dtype)

    def dense(xh, g):
        if layout == "nhwc":
            xh, g = np.ascontiguousarray(xh.transpose(0, 3, 1, 2)), np.ascontiguousarray(g.transpose(0, 3, 1, 2))
        r = oracle.dw_conv(xh, g, kh, kw, (sh, sw), (ph, pw), (dh, dw))
        return r.transpose(0, 2, 3, 1) if layout == "nhwc" else r

    check(x, dy, 0.6, J, dense, shape[0] * OH * OW, conv=geom, layout=layout)


@pytest.mark.parametrize("dtype,layout,shape,J,geom", [
    ("f32", "nchw", (2, 5, 6, 7), 6, (3, 3, 1, 1, 1, 1, 1, 1)), ("f32", "nchw", (3, 40, 9, 12), 130, (3, 3, 1, 1, 1, 1, 1, 1)),
    ("f32", "nchw", (2, 9, 11, 8), 70, (5, 3, 2, 1, 2, 1, 1, 2)), ("f32", "nhwc", (2, 9, 8, 24), 68, (3, 3, 1, 1, 1, 1, 1, 1)),
    ("f32", "nhwc", (2, 7, 10, 6), 5, (3, 3, 2, 2, 1, 1, 1, 1)), ("bf16", "nchw", (2, 9, 13, 10), 12, (5, 3, 1, 2, 2, 1, 1, 1)),
    ("bf16", "nhwc", (2, 8, 6, 16), 9, (3, 3, 1, 1, 2, 2, 2, 2)), ("f32", "nchw", (2, 6, 5, 5), 8, (2, 2, 1, 1, 0, 0, 1, 1))])
def test_infinities_do_not_meet_the_padding(dtype, layout, shape, J, geom):
    """Infinities and NaN of dY, at borders and inside, and of x: a window position over the padding is no term of the sum
    (as in the oracle), so a tap that hangs over the border there stays what the other terms make it."""
    print("exact non-finite", dtype, layout, shape, J, geom, flush=True)
    kh, kw, sh, sw, ph, pw, dh, dw = geom
    H, W = (shape[1], shape[2]) if layout == "nhwc" else (shape[2], shape[3])
    OH, OW = (H + 2 * ph - dh * (kh - 1) - 1) // sh + 1, (W + 2 * pw - dw * (kw - 1) - 1) // sw + 1
    xf = oracle.widen(activation(shape, "normal", 23 + H, dtype)).astype(np.float32)
    g = oracle.widen(gradient((shape[0], J, OH, OW), 0.02, 24 + W, dtype)).astype(np.float32)
    g[0, 1, 0, 0], g[1, 2, OH - 1, OW - 1], g[0, 3, OH // 2, 0] = np.inf, np.nan, -np.inf
    g[1, 4, 0, :] = np.inf
    xf.reshape(-1)[5] = np.inf
    if layout == "nhwc":
        g = np.ascontiguousarray(g.transpose(0, 2, 3, 1))
    x, dy = (xf, g) if dtype == "f32" else (f32_to_bf16_bits(xf), f32_to_bf16_bits(g))
    for gamma in (0.0, 0.5):
        vals, idx = dropit.compress(to_device(x), gamma)
        assert dropit.weight_grad_path(shape, vals.dtype, vals.numel(), J, geom, layout=layout) == "fma"
        got = to_host(dropit.weight_grad(vals, idx, shape, to_device(dy), J, conv=geom, layout=layout)).astype(np.float64)
        xh, yh = oracle.densify(*oracle.compress(x, oracle.keep_count(x.size, gamma)), shape), oracle.widen(dy)
        if layout == "nhwc":
            xh, yh = np.ascontiguousarray(xh.transpose(0, 3, 1, 2)), np.ascontiguousarray(yh.transpose(0, 3, 1, 2))
            got = got.transpose(0, 3, 1, 2)
        ref = oracle.dw_conv(xh, yh, kh, kw, (sh, sw), (ph, pw), (dh, dw))
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).any() and np.isfinite(ref).any()
        inf = np.isinf(ref)
        assert np.array_equal(got[inf], ref[inf])
        fin = np.isfinite(ref)
        size = oracle.dw_conv(np.abs(np.where(np.isfinite(xh), xh, 0)), np.abs(np.where(np.isfinite(yh), yh, 0)), kh, kw, (sh, sw),
                              (ph, pw), (dh, dw))
        nu = (shape[0] * OH * OW + 256) * 2.0 ** -24
        assert (np.abs(got[fin] - ref[fin]) <= nu / (1 - nu) * size[fin]).all()


@pytest.mark.parametrize("dtype,ntok,cin,cout", [("f32", 20000, 12, 4), ("f32", 6304, 384, 260), ("f32", 32001, 61, 67), ("bf16", 9000, 130, 129)])
def test_integer_sums_are_exact(dtype, ntok, cin, cout):
    """Whole numbers of magnitude up to 8, whose sums are exact in fp32 in any order: no term of a long sum left out, taken
    twice or misplaced."""
    print("exact integers", dtype, ntok, cin, cout, flush=True)
    rng = np.random.default_rng(ntok)
    xf, g = rng.integers(-8, 9, (ntok, cin)).astype(np.float32), rng.integers(-8, 9, (ntok, cout)).astype(np.float32)
    x, dy = (xf, g) if dtype == "f32" else (f32_to_bf16_bits(xf), f32_to_bf16_bits(g))
    vals, idx = dropit.compress(to_device(x), 0.4)
    assert dropit.weight_grad_path(x.shape, vals.dtype, vals.numel(), cout) == "fma"
    got = to_host(dropit.weight_grad(vals, idx, x.shape, to_device(dy), cout)).astype(np.float64)
    xh = oracle.densify(*oracle.compress(x, oracle.keep_count(x.size, 0.4)), x.shape)
    assert np.array_equal(got, oracle.widen(dy).astype(np.float64).T @ xh)


@pytest.mark.parametrize("layout,shape,J,geom", [("nchw", (32, 24, 32, 32), 40, (3, 3, 1, 1, 1, 1, 1, 1)),
                                                 ("nhwc", (9, 41, 37, 20), 70, (3, 3, 2, 2, 1, 1, 1, 1))])
def test_integer_convolution_sums_are_exact(layout, shape, J, geom):
    print("exact integer conv", layout, shape, J, geom, flush=True)
    kh, kw, sh, sw, ph, pw, dh, dw = geom
    N, C, H, W = shape if layout == "nchw" else (shape[0], shape[3], shape[1], shape[2])
    OH, OW = (H + 2 * ph - dh * (kh - 1) - 1) // sh + 1, (W + 2 * pw - dw * (kw - 1) - 1) // sw + 1
    rng = np.random.default_rng(H)
    x = rng.integers(-8, 9, shape).astype(np.float32)
    dy = rng.integers(-8, 9, (N, J, OH, OW) if layout == "nchw" else (N, OH, OW, J)).astype(np.float32)
    vals, idx = dropit.compress(to_device(x), 0.4)
    got = to_host(dropit.weight_grad(vals, idx, shape, to_device(dy), J, conv=geom, layout=layout)).astype(np.float64)
    xh, g = oracle.densify(*oracle.compress(x, oracle.keep_count(x.size, 0.4)), shape), dy
    if layout == "nhwc":
        xh, g, got = (np.ascontiguousarray(a.transpose(0, 3, 1, 2)) for a in (xh, g, got))
    assert np.array_equal(got, oracle.dw_conv(xh, g, kh, kw, (sh, sw), (ph, pw), (dh, dw)))


@pytest.mark.parametrize("height,dtype", [(16384, torch.float32), (16383, torch.float32), (32768, torch.bfloat16), (32767, torch.bfloat16)])
def test_either_side_of_32_bit_offsets(height, dtype):
    """Operands of 2 GiB, and just below: 64-bit addresses on one side, buffer descriptors with 32-bit offsets on the other.
    A 1 x 1 convolution of two images and one channel; every sum is of whole numbers below 2^24 per slice, so it is exact up to
    the rounding of the slices' sums."""
    print("exact offsets", height, dtype, flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(height)
    shape = (2, 1, height, 16384)
    x = torch.randint(-3, 4, shape, generator=gen, device="cuda:0", dtype=torch.int8).to(dtype)
    dy = torch.randint(0, 2, shape, generator=gen, device="cuda:0", dtype=torch.int8).to(dtype)
    vals, idx = dropit.compress(x, 0.3)
    got = dropit.weight_grad(vals, idx, shape, dy, 1, conv=(1, 1, 1, 1, 0, 0, 1, 1))
    flat = dy.reshape(-1)
    want = sum((vals[i:i + (1 << 26)].double() * flat[idx[i:i + (1 << 26)].long()].double()).sum().item()
               for i in range(0, vals.numel(), 1 << 26))
    scale = sum((vals[i:i + (1 << 26)].double() * flat[idx[i:i + (1 << 26)].long()].double()).abs().sum().item()
                for i in range(0, vals.numel(), 1 << 26))
    assert got.numel() == 1 and abs(got.item() - want) <= 2.0 ** -22 * scale


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("J", [3, 70])
def test_infinities_of_the_next_image(dtype, J):
    """A tile's rows past the last output channel reach into the next image: an infinity there, at the first channels, is in the
    sums of its own channels alone, padded or not, whichever slices the images are in."""
    print("exact next image", dtype, J, flush=True)
    shape, conv, OH, OW = (24, 5, 15, 17), (3, 3, 2, 2, 1, 1, 1, 1), 8, 9
    x, g = activation(shape, "normal", 31, dtype), oracle.widen(gradient((24, J, OH, OW), 0.02, 32, dtype)).astype(np.float32)
    g[3, 0, 4, 4], g[11, 1, 0, 0], g[23, 0, 7, 8] = np.inf, np.nan, -np.inf
    dy = g if dtype == "f32" else f32_to_bf16_bits(g)
    vals, idx = dropit.compress(to_device(x), 0.5)
    assert dropit.weight_grad_path(shape, vals.dtype, vals.numel(), J, conv) == "fma"
    got = to_host(dropit.weight_grad(vals, idx, shape, to_device(dy), J, conv=conv)).astype(np.float64)
    xh = oracle.densify(*oracle.compress(x, oracle.keep_count(x.size, 0.5)), shape)
    ref = oracle.dw_conv(xh, oracle.widen(dy), 3, 3, (2, 2), (1, 1))
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    assert fin[2:].all() and not fin[:2].all()
    size = oracle.dw_conv(np.abs(xh), np.abs(np.where(np.isfinite(g), oracle.widen(dy), 0)), 3, 3, (2, 2), (1, 1))
    nu = (24 * OH * OW + 256) * 2.0 ** -24
    assert (np.abs(got[fin] - ref[fin]) <= nu / (1 - nu) * size[fin]).all()
