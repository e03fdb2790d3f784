"""GPU: the persistent select's fp32 form -- a bracket from a sample, the threshold's bin exchanged as a list -- at the sizes
and values where it changes over: the smallest tensors, wavefront ranges that end inside a row, more candidates than the LDS
segments hold, a bin of more elements than the list holds (ties, large tensors), a sample that misleads, no usable bracket,
and workgroups that give up: bit for bit against the oracle.  Word 63 of the state block says which way a call went: 0 exact
first digit, 1 bracket confirmed, 2 missed, + 4 where the bin went through a histogram."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


def run(x, gamma, fill=0x5A):
    xd = to_device(x)
    ws = torch.full((dropit.compress_workspace_bytes(x.size, xd.dtype),), fill, dtype=torch.uint8, device="cuda:0")
    k = oracle.keep_count(x.size, gamma)
    want_v, want_i = oracle.compress(x, k)
    vals, idx = dropit.compress(xd, gamma, workspace=ws)
    torch.cuda.synchronize()
    form = int(ws[:256].cpu().numpy().view(np.uint32)[63])
    print("fp32 select", x.size, gamma, "form", form, flush=True)
    assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes(), (x.size, gamma)
    return form


def normal(n, seed=3):
    return np.random.default_rng(seed + n % 101).standard_normal(n, dtype=np.float32)


@pytest.mark.parametrize("numel", [32772, 32775, 4 * (8192 + 64) + 1, 65536, 131075, 300001, 1 << 20, 2420736, (1 << 21) - 5])
def test_sizes(numel):
    for gamma in (0.9, 0.6):
        assert run(normal(numel), gamma) & 3 == 1
    run(normal(numel), 0.05)                           # (small magnitudes: the bracket takes more bins than it may)
    relu = np.maximum(normal(numel), 0)
    assert run(relu, 0.8) & 3 == 1
    run(relu, 0.3)                                     # the threshold is zero: half of the tensor ties there
    assert run(normal(numel), 1.0 - 7.0 / numel) & 3 == 0      # no rank to bracket


def test_segments_overflow():
    """Most elements are candidates: rows are read again for the counts, the list and the output."""
    assert run(normal(9000011), 0.2) & 3 == 1
    run(normal(6000000), 0.02)


def test_large_bin():
    """More than 16384 elements in the threshold's bin: its histogram and a second table."""
    assert run(normal(21000003), 0.9) == 5
    x = np.random.default_rng(1).integers(-4, 5, 400003).astype(np.float32)
    for gamma in (0.9, 0.8, 0.5):
        assert run(x, gamma) & 4 == 4
    run(np.full(100000, -0.75, dtype=np.float32), 0.7)
    run(np.zeros(100000, dtype=np.float32), 0.7)


def test_ties_end_at_any_wavefront():
    numel = 300003
    rng = np.random.default_rng(numel)
    x = rng.standard_normal(numel).astype(np.float32)
    x[rng.permutation(numel)[:9000]] = 1.5             # a list of ties among others
    mag = np.abs(x)
    big, ties = int((mag > 1.5).sum()), int((mag == 1.5).sum())
    for m in (1, 2, ties // 3, ties // 2, ties - 1, ties):
        gamma = 1.0 - (big + m + 0.5) / numel
        assert oracle.keep_count(numel, gamma) == big + m
        assert run(x, gamma) == 1


@pytest.mark.parametrize("numel", [1 << 17, 1 << 21])
@pytest.mark.parametrize("scale", [0.01, 100.0])
def test_misled(numel, scale):
    """The sampled pieces (512 of four vectors, one per stretch at a hashed place) have another scale than the rest."""
    nvf = numel // 4
    stretch = nvf // 4 // 512
    sampled = np.zeros(nvf, dtype=bool)
    for i in range(512):
        first = (i * stretch + ((((i + 1) * 0x9E3779B1) & 0xFFFFFFFF) >> 8) % stretch) * 4
        sampled[first:first + 4] = True
    x = normal(numel) * np.where(np.repeat(sampled, 4), np.float32(scale), np.float32(1.0))
    for gamma in (0.9, 0.5):
        assert run(x, gamma) & 3 == 2


def test_infinities_and_ragged_end():
    x = normal(200003)
    x[::9] = np.inf
    x[4::17] = np.nan
    x[-3:] = [np.nan, -np.inf, 1e-42]
    for gamma in (0.95, 0.9, 0.87, 0.5):
        run(x, gamma)
    x = normal(200003)
    x[-3:] = 1.7                                       # the ragged end near the threshold, in the list
    run(x, 0.9)


@pytest.mark.parametrize("numel", [40001, 300003, 2420736])
def test_without_patience(numel):
    dropit.set_select_mode(3)
    try:
        for fill in range(4):
            run(normal(numel), 0.9, fill)
            run(np.maximum(normal(numel), 0), 0.3, fill)
    finally:
        dropit.set_select_mode(0)


def test_replays():
    """A captured call over changing inputs, eager calls between the replays."""
    n = 300003
    xd = to_device(normal(n))
    k = dropit.keep_count(n, 0.9)
    vals, idx = torch.empty(k, device="cuda:0"), torch.empty(k, dtype=torch.int32, device="cuda:0")
    ws = torch.empty(dropit.compress_workspace_bytes(n, xd.dtype), dtype=torch.uint8, device="cuda:0")
    dropit.compress(xd, 0.9, vals=vals, idx=idx, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dropit.compress(xd, 0.9, vals=vals, idx=idx, workspace=ws)
    for seed in range(5):
        x = normal(n, seed) if seed != 3 else np.random.default_rng(2).integers(-4, 5, n).astype(np.float32)
        xd.copy_(torch.from_numpy(x))
        graph.replay()
        torch.cuda.synchronize()
        want_v, want_i = oracle.compress(x, k)
        assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes()
        run(x, 0.6)
