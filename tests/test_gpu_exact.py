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
from dropit_inputs import activation, gradient
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
