"""GPU: selects on two streams at once, a large tensor and a small one whose few workgroups meet at grid barriers too: whoever finds
the compute units taken by the other gives up after a bounded wait and redoes its selection alone; the bytes are the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import activation
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


def prepared(numel, gamma, dist):
    x = activation((numel,), dist, numel % 97, "bf16")
    k = oracle.keep_count(numel, gamma)
    xd = to_device(x)
    return (xd, gamma, torch.zeros(k, dtype=torch.bfloat16, device="cuda:0"), torch.zeros(k, dtype=torch.int32, device="cuda:0"),
            torch.empty(dropit.compress_workspace_bytes(numel, xd.dtype), dtype=torch.uint8, device="cuda:0"), oracle.compress(x, k))


@pytest.mark.parametrize("numel,gamma", [(30000, 0.6), (60000, 0.6), (49152, 0.9)])
def test_small_beside_large(numel, gamma):
    sides = [(torch.cuda.Stream(), 3, prepared(5000000, 0.9, "gelu")), (torch.cuda.Stream(), 8, prepared(numel, gamma, "normal"))]
    torch.cuda.synchronize()
    for rep in range(60):
        for stream, calls, (xd, g, vals, idx, ws, _) in sides:
            with torch.cuda.stream(stream):
                for _ in range(calls):
                    dropit.compress(xd, g, vals=vals, idx=idx, workspace=ws)
        torch.cuda.synchronize()
        if rep % 10 == 0:
            print("two streams", numel, gamma, rep, flush=True)
            for _, _, (_, _, vals, idx, _, (want_v, want_i)) in sides:
                assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes()
                vals.zero_()
                idx.zero_()
            torch.cuda.synchronize()
