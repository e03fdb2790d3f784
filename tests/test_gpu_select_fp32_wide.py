"""GPU: the fp32 select where its table of 2^16-key bins does not reach: brackets of more than seven sample bins (bins of 2^17 and
2^18 keys, settled by the list alone, with a third digit), a wide bin that turns out to hold more than the list, and thresholds
among the zeros or just above them -- bit for bit against the oracle.  Word 63 of the state block says which way a call went: 0
exact first digit, 1 bracket confirmed, 2 missed, + 4 where the bin held more elements than the list."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


def run(x, gamma):
    xd = to_device(x)
    ws = torch.full((dropit.compress_workspace_bytes(x.size, xd.dtype),), 0x6B, dtype=torch.uint8, device="cuda:0")
    want_v, want_i = oracle.compress(x, oracle.keep_count(x.size, gamma))
    vals, idx = dropit.compress(xd, gamma, workspace=ws)
    torch.cuda.synchronize()
    form = int(ws[:256].cpu().numpy().view(np.uint32)[63])
    print("fp32 wide", x.size, gamma, "form", form, flush=True)
    assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes(), (x.size, gamma)
    return form


@pytest.mark.parametrize("numel", [40004, 150001, 700000, 1500003])
@pytest.mark.parametrize("spread", [2.5, 4.0, 5.0])
def test_wide_brackets(numel, spread):
    """Magnitudes spread over many octaves: brackets of 8 to 28 sample bins."""
    x = np.exp(spread * np.random.default_rng(numel).standard_normal(numel)).astype(np.float32)
    x[::3] *= -1
    for gamma in (0.9, 0.6, 0.3):
        assert run(x, gamma) == 1


def test_rectified():
    for numel, gammas in ((300003, (0.6, 0.7)), (1200000, (0.6, 0.7))):
        x = np.maximum(np.random.default_rng(numel).standard_normal(numel), 0).astype(np.float32)
        for gamma in gammas:
            assert run(x, gamma) == 1


def test_a_wide_bin_of_more_than_the_list_holds():
    """The sampled pieces (512 of four vectors, one per stretch at a hashed place) do not show the value that half of the other
    elements have."""
    numel = 1 << 19
    rng = np.random.default_rng(8)
    x = np.exp(3.0 * rng.standard_normal(numel)).astype(np.float32)
    nvf, other = numel // 4, np.ones(numel // 4, dtype=bool)
    stretch = nvf // 4 // 512
    for i in range(512):
        first = (i * stretch + ((((i + 1) * 0x9E3779B1) & 0xFFFFFFFF) >> 8) % stretch) * 4
        other[first:first + 4] = False
    x[np.repeat(other, 4) & (rng.random(numel) < 0.5)] = 1.0
    assert run(x, 0.5) == 2 + 4


@pytest.mark.parametrize("numel", [40003, 300003, 2420736])
def test_threshold_among_the_zeros(numel):
    rng = np.random.default_rng(numel)
    x = np.maximum(rng.standard_normal(numel), 0).astype(np.float32)
    x[rng.random(numel) < 0.01] = -0.0
    above = int((x != 0).sum())
    for k in (above + 1, above + 1000, numel - 1, numel):
        gamma = 1.0 - (k + (0.5 if k < numel else 0.0)) / numel
        assert oracle.keep_count(numel, gamma) == k
        run(x, gamma)
    run(np.zeros(numel, dtype=np.float32), 0.7)


@pytest.mark.parametrize("numel", [40003, 300003, 2420736])
def test_threshold_just_above_the_zeros(numel):
    """Half zeros, and a fifth subnormal values that share their first digit, few of them or many the same."""
    rng = np.random.default_rng(numel)
    x = rng.standard_normal(numel).astype(np.float32)
    kind = rng.random(numel)
    x[kind < 0.5] = 0.0
    tiny = (kind >= 0.5) & (kind < 0.7)
    for bits in (rng.integers(1, 1 << 18, numel), rng.integers(1, 5, numel), np.full(numel, 70000)):
        x[tiny] = bits.astype(np.uint32).view(np.float32)[tiny]
        large, some = int((np.abs(x) > 1e-30).sum()), int(tiny.sum())
        for k in (large + 1, large + some // 2, large + some, large + some + 1):
            gamma = 1.0 - (k + 0.5) / numel
            assert oracle.keep_count(numel, gamma) == k
            run(x, gamma)


@pytest.mark.parametrize("numel", [33000, 300003, 5000000])
def test_two_tables_in_a_row(numel):
    """A threshold just above the zeros takes two tables, one after the other in the same lines: workgroups with little to stage
    must not write the second before the others have read the first.  All of the work lies in the last workgroups here."""
    x = np.zeros(numel, dtype=np.float32)
    rng = np.random.default_rng(numel)
    some = numel // 8
    x[-some:] = rng.integers(1, 1 << 17, some).astype(np.uint32).view(np.float32)
    k = numel // 16
    gamma = 1.0 - (k + 0.5) / numel
    assert oracle.keep_count(numel, gamma) == k
    want_v, want_i = oracle.compress(x, k)
    xd = to_device(x)
    ws = torch.empty(dropit.compress_workspace_bytes(numel, xd.dtype), dtype=torch.uint8, device="cuda:0")
    for rep in range(40):
        vals, idx = dropit.compress(xd, gamma, workspace=ws)
        torch.cuda.synchronize()
        assert int(ws[:64].cpu().numpy().view(np.uint32)[14]) == 0, rep
        assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes(), rep


def test_without_patience():
    rng = np.random.default_rng(4)
    relu = np.maximum(rng.standard_normal(300003), 0).astype(np.float32)
    dropit.set_select_mode(3)
    try:
        for _ in range(3):
            run(np.exp(4.0 * rng.standard_normal(300003)).astype(np.float32), 0.8)
            run(relu, 0.3)
            run(relu, 0.6)
    finally:
        dropit.set_select_mode(0)
