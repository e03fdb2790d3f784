"""GPU: mode 3 of the select redoes the selection alone on every call, whatever the sizes and however quickly the workgroups meet
at the grid barriers (a grid of one workgroup is always complete when it looks), and says so in word 14 of the state block."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import activation
from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,numel", [("bf16", 13), ("bf16", 5000), ("bf16", 20000), ("bf16", 70000), ("bf16", 600000),
                                         ("f32", 7), ("f32", 4000), ("f32", 33000), ("f32", 300000)])
def test_every_call_without_patience_is_redone(dtype, numel):
    x = activation((numel,), "normal", 3 + numel % 89, dtype)
    want_v, want_i = oracle.compress(x, oracle.keep_count(numel, 0.8))
    xd = to_device(x)
    ws = torch.empty(dropit.compress_workspace_bytes(numel, xd.dtype), dtype=torch.uint8, device="cuda:0")
    dropit.set_select_mode(3)
    try:
        for rep in range(30):
            ws.fill_(rep)
            vals, idx = dropit.compress(xd, 0.8, workspace=ws)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(idx), want_i) and to_host(vals).tobytes() == want_v.tobytes()
            assert int(ws[:64].cpu().numpy().view(np.uint32)[14]) == 1, rep
    finally:
        dropit.set_select_mode(0)
