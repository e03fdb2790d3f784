"""GPU: the row and mask forms written by the select itself (16-bit tensors above 64 K elements without a ragged end), against
the oracle: rows of every kind of length (shorter than a vector, longer than a wavefront's range, one row), blocks and mask
words that end inside a wavefront's range, few and many kept elements, segments that overflow, ties that split a wavefront, a
forced serial redo, a sample that misleads, graph replays, and guard words around what is written."""
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


def misleading(numel, scale):
    """Sampled pieces (512 of two vectors, one per stretch at a hashed place) of another scale than the rest."""
    nvf = numel // 8
    stretch, sampled = nvf // 4 // 512, np.zeros(nvf, dtype=bool)
    for i in range(512):
        first = (i * stretch + ((((i + 1) * 0x9E3779B1) & 0xFFFFFFFF) >> 8) % stretch) * 4
        sampled[first:first + 2] = True
    base = np.random.default_rng(numel).standard_normal(numel, dtype=np.float32)
    return f32_to_bf16_bits(base * np.where(np.repeat(sampled, 8), np.float32(scale), np.float32(1.0)))


@pytest.mark.parametrize("mode", [0, 3])
@pytest.mark.parametrize("scale", [0.01, 100.0])
def test_misled(scale, mode):
    """The retry, which begins when the workgroups have already reported; without patience some give up in it."""
    dropit.set_select_mode(mode)
    try:
        for shape in ((1024, 128), (32768, 64), (1 << 18, 8)):
            check(misleading(shape[0] * shape[1], scale), shape, 0.9)
    finally:
        dropit.set_select_mode(0)


def guarded(words, dtype):
    whole = torch.full((words + 128,), 0x5A5A if dtype == torch.int16 else 0x5A5A5A5A, dtype=dtype, device="cuda:0")
    return whole, whole[64:64 + words]


def intact(whole):
    edge = torch.cat((whole[:64], whole[-64:]))
    return bool((edge == edge[0]).all()) and int(edge[0]) in (0x5A5A, 0x5A5A5A5A)


@pytest.mark.parametrize("shape,gamma", [((8193, 8), 0.9), ((32772, 2), 0.99), ((1000, 1032), 0.6), ((3, 65536), 0.9), ((700003, 8), 0.05),
                                         ((2420, 1000), 0.9)])
@pytest.mark.parametrize("mode", [0, 3])
def test_nothing_is_written_outside_the_outputs(shape, gamma, mode):
    size = int(np.prod(shape))
    x = activation((size,), "gelu", 7 + size % 89, "bf16")
    xd, k = to_device(x).reshape(shape), oracle.keep_count(size, gamma)
    want_v, want_i = oracle.compress(x, k)
    lib, code, dims = dropit.lib(), dropit.binding._dtype_code(xd.dtype), dropit.binding._shape_array(shape)
    stream, rows, blocks = torch.cuda.current_stream().cuda_stream, size // shape[-1], (size + 1023) // 1024
    vals_w, vals = guarded(k, torch.int16)
    col_w, col = guarded(k, torch.int16)
    starts_w, starts = guarded(rows + 1, torch.int32)
    mask_w, mask = guarded((size + 31) // 32, torch.int32)
    block_w, block = guarded(blocks + 1, torch.int32)
    print("index forms guarded", shape, gamma, mode, flush=True)
    dropit.set_select_mode(mode)
    try:
        n = lib.dropit_compress_rows_workspace_bytes(size, k, code)
        ws = torch.full((n,), 0xEE, dtype=torch.uint8, device="cuda:0")
        assert lib.dropit_compress_rows(xd.data_ptr(), dims, 2, code, gamma, vals.data_ptr(), col.data_ptr(), starts.data_ptr(),
                                        ws.data_ptr(), n, stream) == 0
        torch.cuda.synchronize()
        assert intact(vals_w) and intact(col_w) and intact(starts_w)
        assert np.array_equal(col.cpu().numpy().view(np.uint16), (want_i % shape[-1]).astype(np.uint16))
        assert np.array_equal(starts.cpu().numpy(), np.searchsorted(want_i, np.arange(rows + 1, dtype=np.int64) * shape[-1]))
        n = lib.dropit_compress_mask_workspace_bytes(size, k, code)
        ws = torch.full((n,), 0xEE, dtype=torch.uint8, device="cuda:0")
        vals.zero_()
        assert lib.dropit_compress_mask(xd.data_ptr(), dims, 2, code, gamma, vals.data_ptr(), mask.data_ptr(), block.data_ptr(),
                                        ws.data_ptr(), n, stream) == 0
        torch.cuda.synchronize()
    finally:
        dropit.set_select_mode(0)
    assert intact(vals_w) and intact(mask_w) and intact(block_w)
    assert vals.cpu().numpy().view(np.uint16).tobytes() == want_v.tobytes()
    bits = np.zeros((size + 31) // 32 * 32, dtype=np.uint8)
    bits[want_i] = 1
    assert np.array_equal(mask.cpu().numpy().view(np.uint32), np.packbits(bits, bitorder="little").view(np.uint32))
    assert np.array_equal(block.cpu().numpy(), np.searchsorted(want_i, np.arange(blocks + 1, dtype=np.int64) * 1024))


def test_replays():
    """Captured calls of both forms over changing inputs, eager calls between the replays."""
    shape, gamma = (3000, 104), 0.9
    size = shape[0] * shape[1]
    k, code, dims = oracle.keep_count(size, gamma), dropit.binding.BF16, dropit.binding._shape_array(shape)
    lib, blocks = dropit.lib(), (size + 1023) // 1024
    xd = to_device(activation((size,), "normal", 1, "bf16")).reshape(shape)
    dev = xd.device
    vals_r, vals_m = (torch.empty(k, dtype=torch.bfloat16, device=dev) for _ in range(2))
    col, starts = torch.empty(k, dtype=torch.int16, device=dev), torch.empty(shape[0] + 1, dtype=torch.int32, device=dev)
    mask, block = torch.empty((size + 31) // 32, dtype=torch.int32, device=dev), torch.empty(blocks + 1, dtype=torch.int32, device=dev)
    nr, nm = lib.dropit_compress_rows_workspace_bytes(size, k, code), lib.dropit_compress_mask_workspace_bytes(size, k, code)
    ws_r, ws_m = torch.empty(nr, dtype=torch.uint8, device=dev), torch.empty(nm, dtype=torch.uint8, device=dev)

    def both():
        stream = torch.cuda.current_stream().cuda_stream
        assert lib.dropit_compress_rows(xd.data_ptr(), dims, 2, code, gamma, vals_r.data_ptr(), col.data_ptr(), starts.data_ptr(),
                                        ws_r.data_ptr(), nr, stream) == 0
        assert lib.dropit_compress_mask(xd.data_ptr(), dims, 2, code, gamma, vals_m.data_ptr(), mask.data_ptr(), block.data_ptr(),
                                        ws_m.data_ptr(), nm, stream) == 0

    both()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        both()
    for replay, dist in enumerate(("gelu", "normal", "relu", "gelu", "normal")):
        x = activation((size,), dist, 60 + replay, "bf16")
        xd.copy_(to_device(x).reshape(shape))
        for t in (vals_r, vals_m, col, starts, mask, block):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want_v, want_i = oracle.compress(x, k)
        assert to_host(vals_r).tobytes() == want_v.tobytes() and to_host(vals_m).tobytes() == want_v.tobytes(), replay
        assert np.array_equal(col.cpu().numpy().view(np.uint16), (want_i % shape[1]).astype(np.uint16))
        assert np.array_equal(starts.cpu().numpy(), np.searchsorted(want_i, np.arange(shape[0] + 1, dtype=np.int64) * shape[1]))
        bits = np.zeros((size + 31) // 32 * 32, dtype=np.uint8)
        bits[want_i] = 1
        assert np.array_equal(mask.cpu().numpy().view(np.uint32), np.packbits(bits, bitorder="little").view(np.uint32))
        assert np.array_equal(block.cpu().numpy(), np.searchsorted(want_i, np.arange(blocks + 1, dtype=np.int64) * 1024))
        check(activation((200000,), dist, replay, "bf16"), (200, 1000), 0.8)
