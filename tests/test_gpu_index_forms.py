"""GPU: the row and mask forms written by the select itself (16-bit tensors above 64 K elements without a ragged end), against
the oracle: rows of every kind of length (shorter than a vector, longer than a wavefront's range, one row), blocks and mask
words that end inside a wavefront's range, few and many kept elements, segments that overflow, ties that split a wavefront, a
forced serial redo and graph replays."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import activation, f32_to_bf16_bits
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


def check(x, shape, gamma):
    xd = to_device(x).reshape(shape)
    k = oracle.keep_count(x.size, gamma)
    want_v, want_i = oracle.compress(x, k)
    print("index forms", shape, gamma, k, flush=True)
    length = shape[-1]
    if length <= 65536:
        vals, col, rowptr = dropit.compress_rows(xd, gamma)
        torch.cuda.synchronize()
        assert to_host(vals).tobytes() == want_v.tobytes()
        assert np.array_equal(to_host(col).view(np.uint16), (want_i % length).astype(np.uint16))
        rows = x.size // length
        assert np.array_equal(to_host(rowptr), np.searchsorted(want_i, np.arange(rows + 1, dtype=np.int64) * length))
    vals, mask, blockptr = dropit.compress_mask(xd, gamma)
    torch.cuda.synchronize()
    assert to_host(vals).tobytes() == want_v.tobytes()
    bits = np.zeros((x.size + 31) // 32 * 32, dtype=np.uint8)
    bits[want_i] = 1
    assert np.array_equal(to_host(mask).view(np.uint32), np.packbits(bits, bitorder="little").view(np.uint32))
    blocks = (x.size + 1023) // 1024
    assert np.array_equal(to_host(blockptr), np.searchsorted(want_i, np.arange(blocks + 1, dtype=np.int64) * 1024))


@pytest.mark.parametrize("shape", [
    (65544,), (32772, 2), (9000, 8), (12345, 24), (1000, 1032), (257, 4000), (3, 65536), (8, 50000), (700003, 8), (2420, 1000),
])
def test_shapes(shape):
    size = int(np.prod(shape))
    for gamma, dist in ((0.9, "normal"), (0.6, "gelu"), (0.995, "normal"), (0.05, "relu")):
        check(activation((size,), dist, 3 + size % 97, "bf16"), shape, gamma)


def test_little_is_kept():
    """A handful of elements in a large tensor: windows of nothing but zero words, rows without elements."""
    x = np.zeros(3000000, dtype=np.uint16)
    x[[5, 1023, 1024, 777777, 2999999]] = 0x4000
    for shape in ((3000, 1000), (375000, 8)):
        check(x, shape, 1.0 - 4.5 / x.size)
        check(x, shape, 1.0 - 1.5 / x.size)
    check(f32_to_bf16_bits(np.random.default_rng(0).standard_normal(4000000, dtype=np.float32)), (4000, 1000), 0.9999)


def test_segments_overflow_and_ties():
    check(activation((10000000,), "normal", 5, "bf16"), (10000, 1000), 0.05)
    rng = np.random.default_rng(9)
    x = f32_to_bf16_bits(rng.choice(np.array([0.5, -0.5, 1.0, -2.0, 0.0], dtype=np.float32), size=300000))
    big, ties = int(((x & 0x7FFF) > 0x3F00).sum()), int(((x & 0x7FFF) == 0x3F00).sum())
    for m in (1, ties // 3, ties - 1, ties):
        check(x, (300, 1000), 1.0 - (big + m + 0.5) / x.size)


def test_serial_redo():
    dropit.set_select_mode(3)
    try:
        check(activation((200000,), "gelu", 1, "bf16"), (200, 1000), 0.9)
        check(activation((200000,), "gelu", 2, "bf16"), (25000, 8), 0.99)
    finally:
        dropit.set_select_mode(0)


@pytest.mark.parametrize("shape", [(65537,), (16384, 4), (100, 1001)])
def test_converted(shape):
    """One workgroup, or a ragged end: flat indices, converted."""
    check(activation((int(np.prod(shape)),), "normal", 8, "bf16"), shape, 0.9)
