"""GPU: the forms of the persistent select for 16-bit tensors at the sizes and densities where they change over -- the
smallest tensors it takes, wavefront ranges that end inside a row of 512 elements, staging segments that overflow (part of
the tensor is read twice), and ties whose budget runs out inside one wavefront -- bit for bit against the oracle."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import activation, f32_to_bf16_bits
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


def run(x, gamma):
    xd = to_device(x)
    ws = torch.full((dropit.compress_workspace_bytes(x.size, xd.dtype),), 0x5A, dtype=torch.uint8, device="cuda:0")
    k = oracle.keep_count(x.size, gamma)
    want_v, want_i = oracle.compress(x, k)
    vals, idx = dropit.compress(xd, gamma, workspace=ws)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes(), (x.size, gamma)
    state = ws[:64].cpu().numpy().view(np.uint32)
    return int(state[10] & 0xFFFF), int(state[15])          # workgroups, those that read the tensor once


@pytest.mark.parametrize("numel", [65544, 65551, 8 * (8192 + 64) + 3, 131072, 300001, 524288 + 8 * 65, 1 << 20, (1 << 21) - 5])
@pytest.mark.parametrize("dist", ["normal", "relu", "gelu"])
def test_mid_sizes(numel, dist):
    x = activation((numel,), dist, 3 + numel % 101, "bf16")
    for gamma in (0.9, 0.6, 0.999, 0.02):
        print("select mid", numel, dist, gamma, run(x, gamma), flush=True)


@pytest.mark.parametrize("numel,gamma", [(9000011, 0.05), (12000000, 0.3), (4 * (1 << 20) + 8 * 333, 0.0)])
def test_segments_overflow(numel, gamma):
    """More candidates than the staging segments hold in (nearly) every workgroup."""
    groups, once = run(activation((numel,), "normal", 5, "bf16"), gamma)
    print("select overflow", numel, gamma, groups, once, flush=True)
    assert groups > 1 and (once < groups or numel < 7800000)


@pytest.mark.parametrize("numel", [300003, (1 << 21) + 777])
def test_tie_budget_runs_out_at_any_wavefront(numel):
    """A handful of magnitudes, so that the kept ties end in the first, a middle and the last wavefronts of the tensor."""
    rng = np.random.default_rng(numel)
    x = f32_to_bf16_bits(rng.choice(np.array([0.5, -0.5, 1.0, -2.0, 0.0], dtype=np.float32), size=numel))
    mag = (x & 0x7FFF)
    big = int((mag > 0x3F00).sum())
    ties = int((mag == 0x3F00).sum())
    for m in (1, 2, ties // 3, ties // 2, ties - 1, ties):
        gamma = 1.0 - (big + m + 0.5) / numel
        assert oracle.keep_count(numel, gamma) == big + m
        run(x, gamma)


def misleading(numel, scale, seed=99):
    """A tensor whose sampled pieces (512 of them, two vectors each, one per equal stretch at a hashed place) have another
    scale than the rest.  numel: a power of two, so that the stretches are equal."""
    nvf = numel // 8
    seg = nvf // 4 // 512
    sampled = np.zeros(nvf, dtype=bool)
    for i in range(512):
        first = (i * seg + ((((i + 1) * 0x9E3779B1) & 0xFFFFFFFF) >> 8) % seg) * 4
        sampled[first:first + 2] = True
    base = np.random.default_rng(seed).standard_normal(numel, dtype=np.float32)
    return f32_to_bf16_bits(base * np.where(np.repeat(sampled, 8), np.float32(scale), np.float32(1.0)))


def form_of(x, gamma):
    """White box: word 8 of the state block, 0 exact digit histograms, 1 sampled bracket confirmed, 2 missed."""
    xd = to_device(x)
    ws = torch.full((dropit.compress_workspace_bytes(x.size, xd.dtype),), 0x33, dtype=torch.uint8, device="cuda:0")
    want_v, want_i = oracle.compress(x, oracle.keep_count(x.size, gamma))
    vals, idx = dropit.compress(xd, gamma, workspace=ws)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes()
    return int(ws[:64].cpu().numpy().view(np.uint32)[8])


@pytest.mark.parametrize("numel", [1 << 17, 1 << 19, 1 << 20, 1 << 22])
def test_prediction_confirmed_and_missed(numel):
    """Below 2 M elements too: a bracket that holds, one that does not (both ways), a quantile without one, fp32."""
    base = np.random.default_rng(7).standard_normal(numel, dtype=np.float32)
    assert form_of(f32_to_bf16_bits(base), 0.9) == 1
    assert form_of(f32_to_bf16_bits(base), 0.99999) == 0
    for gamma in (0.9, 0.5):
        assert form_of(misleading(numel, 0.01), gamma) == 2
        assert form_of(misleading(numel, 100.0), gamma) == 2
    assert form_of(base, 0.9) == 0
    for gamma in (0.05, 0.4):                          # the threshold is zero: half of the tensor ties there
        assert form_of(f32_to_bf16_bits(np.maximum(base, 0)), gamma) == 1
    assert form_of(np.zeros(numel, dtype=np.uint16), 0.7) == 1


@pytest.mark.parametrize("numel", [65552, 70000, 32 * (512 * 5 - 1) + 17, 32 * (512 * 7 - 3), 300001])
def test_sample_covers_the_whole_tensor(numel):
    """Magnitudes that grow with the index, at sizes whose 64-byte places do not divide into 512 equal stretches: the
    sample reaches the end of the tensor, so the prediction holds."""
    x = f32_to_bf16_bits(np.sqrt(np.linspace(0.0, 4.0, numel, dtype=np.float32)))
    for gamma in (0.9, 0.8, 0.5):
        print("stretches", numel, gamma, flush=True)
        assert form_of(x, gamma) == 1


@pytest.mark.parametrize("numel", [1 << 17, 1 << 18, 1 << 21, 1 << 23])
@pytest.mark.parametrize("scale", [0.01, 100.0])
def test_misled_without_patience(numel, scale):
    """A sample that misleads together with workgroups that give up at the grid barriers (mode 3): those that got past the
    first barrier enter the exact form, whose histogram the others no longer publish.  Every wait ends, in milliseconds,
    and the bytes are the oracle's."""
    x = misleading(numel, scale)
    want_v, want_i = oracle.compress(x, oracle.keep_count(numel, 0.9))
    xd = to_device(x)
    ws = torch.empty(dropit.compress_workspace_bytes(numel, xd.dtype), dtype=torch.uint8, device="cuda:0")
    dropit.set_select_mode(3)
    try:
        for rep in range(12):
            print("misled", numel, scale, rep, flush=True)
            ws.fill_(rep)
            torch.cuda.synchronize()
            start = time.perf_counter()
            vals, idx = dropit.compress(xd, 0.9, workspace=ws)
            torch.cuda.synchronize()
            assert time.perf_counter() - start < 0.5
            assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes()
    finally:
        dropit.set_select_mode(0)
