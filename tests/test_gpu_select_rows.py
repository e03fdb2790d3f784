"""GPU: the one-workgroup select by rows of 1024 vectors, at the edges of its rows and of the sizes and kept shares at which other
forms take over (16-bit: 2 and 3 rows, an eighth kept; fp32: 1, 2, 4 and 8 rows, three eighths kept), bit for bit against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import f32_to_bf16_bits
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["normal", "relu", "few"])
@pytest.mark.parametrize("dtype,numel", [
    ("bf16", 8192), ("bf16", 8200), ("bf16", 16391), ("bf16", 16392), ("bf16", 20003), ("bf16", 24576), ("bf16", 24583), ("bf16", 24584),
    ("f32", 2), ("f32", 4096), ("f32", 4099), ("f32", 4100), ("f32", 8195), ("f32", 8196), ("f32", 16387), ("f32", 16388), ("f32", 20480),
    ("f32", 20484), ("f32", 32768), ("f32", 32771)])
def test_edges(dtype, numel, kind):
    x = np.random.default_rng(numel).standard_normal(numel).astype(np.float32)
    x = np.maximum(x, 0) if kind == "relu" else np.round(2 * x) if kind == "few" else x
    x = f32_to_bf16_bits(x) if dtype == "bf16" else x
    xd = to_device(x)
    for kept in (1.0, 0.7, 0.4, 3 / 8, 0.3, 1 / 8, 0.1):
        for k in sorted({int(kept * numel), min(int(kept * numel) + 1, numel)} - {0}):
            gamma = 1.0 - (k + (0.5 if k < numel else 0.0)) / numel
            assert oracle.keep_count(numel, gamma) == k
            want_v, want_i = oracle.compress(x, k)
            vals, idx = dropit.compress(xd, gamma)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes(), (dtype, numel, kind, k)
