"""GPU: the forms of the bf16 convolution gradient that keep no im2col rows, at the edges of their tiles and segments,
element by element against the fp64 product of the recovered tensor.

Bound per element: the products of bf16 numbers are exact in fp32, and an fp32 sum of n of them, in any order and with
any grouping, is within n * 2^-24 of the exact sum relative to the sum of the terms' magnitudes.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import activation, f32_to_bf16_bits, gradient
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu

POINT = (1, 1, 1, 1, 0, 0, 1, 1)


def dense_dw(xh, g, geom):
    """dW [J][C][kh][kw] of NCHW operands in fp64, a tap at a time."""
    kh, kw, sh, sw, ph, pw, dh, dw = geom
    N, C, H, W = xh.shape
    _, J, OH, OW = g.shape
    xp = np.zeros((N, C, H + 2 * ph, W + 2 * pw))
    xp[:, :, ph:ph + H, pw:pw + W] = xh
    flat = np.ascontiguousarray(g.transpose(1, 0, 2, 3)).reshape(J, -1).astype(np.float64)
    out = np.zeros((J, C, kh, kw))
    for u in range(kh):
        for v in range(kw):
            win = xp[:, :, u * dh:u * dh + (OH - 1) * sh + 1:sh, v * dw:v * dw + (OW - 1) * sw + 1:sw]
            out[:, :, u, v] = flat @ np.ascontiguousarray(win.transpose(1, 0, 2, 3)).reshape(C, -1).T
    return out


def check(x, dy, gamma, J, geom, layout="nchw"):
    xd, dyd = to_device(x), to_device(dy)
    vals, idx = dropit.compress(xd, gamma)
    dW = dropit.weight_grad(vals, idx, x.shape, dyd, J, conv=geom, layout=layout)
    again = dropit.weight_grad(vals, idx, x.shape, dyd, J, conv=geom, layout=layout)
    torch.cuda.synchronize()
    assert torch.equal(dW, again)
    xh = oracle.densify(*oracle.compress(x, oracle.keep_count(x.size, gamma)), x.shape)
    g = oracle.widen(dy)
    if layout == "nhwc":
        xh, g = xh.transpose(0, 3, 1, 2), g.transpose(0, 3, 1, 2)
    ref, size = dense_dw(xh, g, geom), dense_dw(np.abs(xh), np.abs(g), geom)
    got = to_host(dW).astype(np.float64)
    if layout == "nhwc":
        got = got.transpose(0, 3, 1, 2)
    nu = (g.shape[0] * g.shape[2] * g.shape[3] + 256) * 2.0 ** -24     # the terms of a sum, and the slices that meet in it
    excess = np.abs(got - ref) - nu / (1 - nu) * size
    assert excess.max() <= 0.0, excess.max()


@pytest.mark.parametrize("shape,J,gamma", [
    ((1, 3, 4, 4), 8, 0.6), ((9, 65, 4, 8), 72, 0.9), ((17, 64, 6, 6), 64, 0.7),      # many planes to a unit, one of them not full
    ((3, 63, 14, 14), 136, 0.8), ((2, 24, 15, 34), 264, 0.8),                           # rows of dY at 8- and 4-byte boundaries
    ((2, 130, 16, 32), 520, 0.9), ((1, 16, 27, 38), 40, 0.9),                           # one and three segments; output channels in two blocks
    ((2, 40, 56, 56), 64, 0.5), ((1, 8, 64, 130), 16, 0.95)])
def test_pointwise_nchw(shape, J, gamma):
    print("pointwise", shape, J, gamma, flush=True)
    x = activation(shape, "relu", 31 + shape[2], "bf16")
    check(x, gradient((shape[0], J, shape[2], shape[3]), 0.02, 32 + J, "bf16"), gamma, J, POINT)


@pytest.mark.parametrize("shape", [(3, 70, 28, 28), (9, 16, 8, 8)])
def test_pointwise_with_crowded_channels(shape):
    """Runs many times longer than an even spread gives, beside empty ones."""
    print("pointwise crowded", shape, flush=True)
    rng = np.random.default_rng(5)
    x = (rng.standard_normal(shape) * 0.01).astype(np.float32)
    x[:, ::9] += 4.0
    x[1, 3] = 0.0
    check(f32_to_bf16_bits(x), gradient((shape[0], 24, shape[2], shape[3]), 0.02, 33, "bf16"), 0.85, 24, POINT)


@pytest.mark.parametrize("shape,J,geom", [
    ((5, 3, 4, 8), 8, (3, 3, 1, 1, 1, 1, 1, 1)), ((40, 1, 5, 24), 136, (1, 3, 1, 1, 0, 1, 1, 1)),     # planes below a token block of 32
    ((7, 9, 9, 40), 264, (3, 3, 1, 1, 1, 1, 1, 1)), ((3, 33, 29, 16), 40, (3, 3, 2, 2, 1, 1, 1, 1)),
    ((2, 20, 31, 72), 144, (5, 3, 1, 2, 2, 3, 1, 2)), ((1, 17, 64, 8), 64, (7, 7, 2, 1, 3, 0, 2, 3)),
    ((2, 6, 6, 512), 128, (3, 3, 1, 1, 2, 2, 2, 2)), ((1, 8, 40, 24), 520, (3, 3, 1, 1, 0, 0, 1, 1)),
    ((64, 14, 14, 64), 64, (3, 3, 1, 1, 1, 1, 1, 1))])
def test_channels_last_window(shape, J, geom):
    print("window nhwc", shape, J, geom, flush=True)
    N, H, W, C = shape
    kh, kw, sh, sw, ph, pw, dh, dw = geom
    OH, OW = (H + 2 * ph - dh * (kh - 1) - 1) // sh + 1, (W + 2 * pw - dw * (kw - 1) - 1) // sw + 1
    x = activation(shape, "relu", 41 + H, "bf16")
    assert dropit.weight_grad_path(shape, torch.bfloat16, x.size // 4, J, geom, layout="nhwc") == "conv_im2col"
    check(x, gradient((N, OH, OW, J), 0.02, 42 + W, "bf16"), 0.7, J, geom, layout="nhwc")


@pytest.mark.parametrize("shape,J", [((33, 128, 14, 14), 128), ((64, 136, 7, 7), 264), ((17, 200, 13, 15), 136),
                                     ((9, 128, 16, 16), 136)])
def test_small_planes_token_major(shape, J):
    print("small planes", shape, J, flush=True)
    geom = (3, 3, 1, 1, 1, 1, 1, 1)
    x = activation(shape, "relu", 51 + shape[1], "bf16")
    assert dropit.weight_grad_path(shape, torch.bfloat16, x.size // 4, J, geom) == "conv_gemm"
    check(x, gradient((shape[0], J, shape[2], shape[3]), 0.02, 52 + J, "bf16"), 0.75, J, geom)


@pytest.mark.parametrize("gamma", [0.0, 0.6, 0.99])
@pytest.mark.parametrize("shape,J,geom", [((4, 96, 21, 3), 16, (3, 3, 1, 1, 0, 0, 1, 1)), ((3, 40, 16, 19), 24, (3, 3, 2, 2, 0, 0, 1, 1)),
                                          ((2, 24, 9, 130), 8, (3, 3, 1, 1, 1, 1, 1, 1))])
def test_sparse_and_full_rows(shape, J, geom, gamma):
    """Row starts with one pair per thread (fewer than eight pairs to a row) and with eight."""
    print("row starts", shape, gamma, flush=True)
    N, C, H, W = shape
    kh, kw, sh, sw, ph, pw, dh, dw = geom
    OH, OW = (H + 2 * ph - dh * (kh - 1) - 1) // sh + 1, (W + 2 * pw - dw * (kw - 1) - 1) // sw + 1
    x = activation(shape, "relu", 61 + H, "bf16")
    check(x, gradient((N, J, OH, OW), 0.02, 62 + W, "bf16"), gamma, J, geom)


@pytest.mark.parametrize("shape,J,geom", [
    ((3, 17, 21, 40), 24, (3, 3, 4, 4, 1, 1, 1, 1)), ((2, 20, 33, 128), 16, (2, 2, 3, 3, 0, 0, 1, 1)),
    ((2, 31, 18, 24), 40, (3, 5, 5, 4, 1, 2, 1, 1)), ((5, 12, 16, 64), 8, (1, 1, 2, 2, 0, 0, 1, 1))])
def test_channels_last_written_rows(shape, J, geom):
    """Channels-last windows whose rows hold less than the input does keep the written rows: several blocks of taps, the
    last one not full."""
    print("rows nhwc", shape, J, geom, flush=True)
    N, H, W, C = shape
    kh, kw, sh, sw, ph, pw, dh, dw = geom
    OH, OW = (H + 2 * ph - dh * (kh - 1) - 1) // sh + 1, (W + 2 * pw - dw * (kw - 1) - 1) // sw + 1
    assert OH * OW * kh * kw < H * W
    x = activation(shape, "relu", 71 + H, "bf16")
    for gamma in (0.3, 0.9):
        check(x, gradient((N, OH, OW, J), 0.02, 72 + W, "bf16"), gamma, J, geom, layout="nhwc")


def integers(shape, seed, zeros):
    """Whole numbers of magnitude up to 8: any sum of fewer than 2^18 of their products is exact in fp32."""
    rng = np.random.default_rng(seed)
    return f32_to_bf16_bits((rng.integers(-8, 9, shape) * (rng.random(shape) >= zeros)).astype(np.float32))


@pytest.mark.parametrize("layout,shape,J,geom", [
    ("nchw", (9, 65, 28, 28), 72, POINT), ("nchw", (2, 40, 56, 56), 64, POINT), ("nchw", (64, 24, 14, 14), 264, POINT),
    ("nhwc", (64, 14, 14, 64), 64, (3, 3, 1, 1, 1, 1, 1, 1)), ("nhwc", (5, 29, 40, 72), 136, (3, 3, 1, 1, 1, 1, 1, 1)),
    ("nhwc", (9, 31, 29, 24), 40, (3, 3, 2, 2, 1, 1, 1, 1)), ("nhwc", (2, 33, 41, 128), 16, (2, 2, 3, 3, 0, 0, 1, 1)),
    ("nchw", (33, 128, 14, 14), 128, (3, 3, 1, 1, 1, 1, 1, 1)), ("nchw", (64, 136, 7, 7), 264, (3, 3, 1, 1, 1, 1, 1, 1)),
    ("nchw", (9, 128, 16, 16), 136, (3, 3, 1, 1, 1, 1, 1, 1)), ("nchw", (7, 40, 28, 30), 24, (3, 3, 1, 1, 1, 1, 1, 1)),
    ("nchw", (11, 24, 33, 31), 16, (3, 3, 2, 2, 1, 1, 1, 1))])
def test_integer_sums_are_exact(layout, shape, J, geom):
    """No term left out, taken twice or misplaced, at sizes of many slices: the sums are whole numbers and must be equal."""
    print("integers", layout, shape, J, geom, flush=True)
    kh, kw, sh, sw, ph, pw, dh, dw = geom
    N, C, H, W = shape if layout == "nchw" else (shape[0], shape[3], shape[1], shape[2])
    OH, OW = (H + 2 * ph - dh * (kh - 1) - 1) // sh + 1, (W + 2 * pw - dw * (kw - 1) - 1) // sw + 1
    x, dy = integers(shape, 81, 0.3), integers((N, J, OH, OW) if layout == "nchw" else (N, OH, OW, J), 82, 0.0)
    vals, idx = dropit.compress(to_device(x), 0.45)
    got = to_host(dropit.weight_grad(vals, idx, shape, to_device(dy), J, conv=geom, layout=layout)).astype(np.float64)
    xh, g = oracle.densify(*oracle.compress(x, oracle.keep_count(x.size, 0.45)), shape), oracle.widen(dy)
    if layout == "nhwc":
        xh, g, got = xh.transpose(0, 3, 1, 2), g.transpose(0, 3, 1, 2), got.transpose(0, 3, 1, 2)
    assert np.array_equal(got, dense_dw(xh, g, geom))


@pytest.mark.parametrize("shape,J", [((2, 512, 14, 14), 512), ((1, 520, 16, 16), 520)])
def test_small_planes_in_one_slice(shape, J):
    """Many tiles and few tokens: the product runs in one slice, which the channel-major order still takes through the
    partial tiles."""
    geom = (3, 3, 1, 1, 1, 1, 1, 1)
    print("one slice", shape, J, flush=True)
    N, C, H, W = shape
    x, dy = integers(shape, 83, 0.3), integers((N, J, H, W), 84, 0.0)
    k = oracle.keep_count(x.size, 0.45)
    assert dropit.weight_grad_path(shape, torch.bfloat16, k, J, geom) == "conv_gemm"
    up = lambda n: (n + 255) // 256 * 256
    tiles = ((9 * C + 255) // 256) * ((J + 255) // 256)
    need = dropit.weight_grad_workspace_bytes(shape, torch.bfloat16, k, J, geom)
    assert need == up((N * H * W + 1) * C * 2) + tiles * 256 * 256 * 4 + up(N * H * W * J * 2)       # one partial tile per tile
    vals, idx = dropit.compress(to_device(x), 0.45)
    got = to_host(dropit.weight_grad(vals, idx, shape, to_device(dy), J, conv=geom)).astype(np.float64)
    xh = oracle.densify(*oracle.compress(x, k), shape)
    assert np.array_equal(got, dense_dw(xh, oracle.widen(dy), geom))
