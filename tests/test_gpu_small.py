"""GPU: the one-launch forms of small tensors and layers at the sizes where they change over -- one vector per thread, the
smallest sampled tensor, the largest of each form, ragged ends, more candidates than the LDS segments hold, and magnitudes
that crowd one histogram bin -- bit for bit against the oracle, and the product against 64 bits."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import f32_to_bf16_bits
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


def values(kind, n, dtype):
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "relu":
        x = np.maximum(x, 0)
    elif kind == "const":
        x = np.full(n, -0.75, dtype=np.float32)
    elif kind == "few":
        x = rng.integers(-4, 5, n).astype(np.float32)
    elif kind == "sorted":
        x = np.linspace(-3, 1, n).astype(np.float32)
    elif kind == "periodic":                       # magnitudes that follow the place in a vector: a fixed place would mislead
        x = x * np.where(np.arange(n) % 8 == 3, 100.0, 1.0).astype(np.float32)
    elif kind == "extreme":
        x[::7] = np.inf
        x[3::11] = np.nan
        x[5::13] = 1e-42                           # a denormal (fp32), zero (bf16)
    return f32_to_bf16_bits(x) if dtype == "bf16" else x


@pytest.mark.parametrize("kind", ["normal", "relu", "const", "few", "sorted", "periodic", "extreme"])
@pytest.mark.parametrize("dtype,numel", [
    ("bf16", 5), ("bf16", 8192), ("bf16", 8199), ("bf16", 8200), ("bf16", 16383), ("bf16", 16384), ("bf16", 32775),
    ("bf16", 32776), ("bf16", 65543),
    ("f32", 3), ("f32", 4099), ("f32", 8191), ("f32", 8192), ("f32", 16384), ("f32", 18443), ("f32", 32771),
])
def test_select(kind, dtype, numel):
    x = values(kind, numel, dtype)
    xd = to_device(x)
    for gamma in (0.0, 0.3, 0.6, 0.9, 0.999, 1.0 - 1.0 / numel):
        k = oracle.keep_count(numel, gamma)
        print("small select", kind, dtype, numel, gamma, k, flush=True)
        if k == 0:
            continue
        want_v, want_i = oracle.compress(x, k)
        vals, idx = dropit.compress(xd, gamma)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(idx), want_i)
        assert to_host(vals).tobytes() == want_v.tobytes()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("ntok,cin,cout", [
    (1, 16384, 5),            # no tokens to share out, four passes of a workgroup over the columns
    (7, 24, 4), (8, 24, 6),   # just below and at two shares
    (128, 128, 130),          # eight shares
    (1024, 16, 33),           # sixteen
    (1024, 4, 2048),          # little work: sixteen rows to a workgroup
    (1024, 12, 2048),         # the most workgroups of four rows
    (31, 20, 2049),           # sixteen rows to a workgroup, the last one nearly empty
    (4, 4096, 2100),
])
def test_layer(dtype, ntok, cin, cout):
    gen = torch.Generator(device="cuda:0").manual_seed(ntok + cout)
    x = torch.randn(ntok, cin, generator=gen, device="cuda:0").to(dtype)
    dy = torch.randn(ntok, cout, generator=gen, device="cuda:0").to(dtype)
    for gamma in (0.0, 0.9):
        vals, idx = dropit.compress(x, gamma)
        assert dropit.weight_grad_path(x.shape, dtype, vals.numel(), cout) == "fc_small"
        flat = torch.zeros(x.numel(), dtype=torch.float64, device="cuda:0")
        flat[idx.long()] = vals.double()
        want = dy.double().t() @ flat.view(ntok, cin)
        got = dropit.weight_grad(vals, idx, x.shape, dy, cout)
        err = ((got.double() - want).norm() / want.norm().clamp(min=1e-30)).item()
        print("small layer", dtype, ntok, cin, cout, gamma, "%.2e" % err, flush=True)
        assert err < 1e-6     # products of fp32 values rounded once, 1024 of them added: 2^-24 sqrt(1024) in the worst direction
