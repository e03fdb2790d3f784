"""GPU: the row form's positions written to an array that starts between 16-byte boundaries (two-byte stores), and to
one that does not, with pair counts around whole groups of eight: the same bits from both."""
import pytest
import torch

import paper_2202_13808_amd as dropit
from dropit_inputs import activation
from gpu_util import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,k", [((65, 24), 8), ((65, 24), 777), ((3, 1), 2), ((40, 65536), 262144), ((7, 5), 35)])
def test_positions_at_any_alignment(shape, k):
    print("rows alignment", shape, k, flush=True)
    x = to_device(activation(shape, "normal", 61, "bf16"))
    gamma = 1.0 - (k + 0.25) / x.numel() if k < x.numel() else 0.0
    vals, col, rowptr = dropit.compress_rows(x, gamma)
    assert vals.numel() == k
    lib, code = dropit.lib(), dropit.binding._dtype_code(x.dtype)
    ws = torch.empty(int(lib.dropit_compress_rows_workspace_bytes(x.numel(), k, code)), dtype=torch.uint8, device=x.device)
    for shift in (1, 4):
        room = torch.full((k + 16,), -1, dtype=torch.int16, device=x.device)
        v2, r2 = torch.empty_like(vals), torch.empty_like(rowptr)
        st = lib.dropit_compress_rows(x.data_ptr(), dropit.binding._shape_array(x.shape), x.dim(), code, float(gamma),
                                      v2.data_ptr(), room[shift:].data_ptr(), r2.data_ptr(), ws.data_ptr(), ws.numel(),
                                      torch.cuda.current_stream().cuda_stream)
        assert st == 0
        torch.cuda.synchronize()
        assert torch.equal(room[shift:shift + k], col) and torch.equal(v2, vals) and torch.equal(r2, rowptr)
        assert bool((room[:shift] == -1).all()) and bool((room[shift + k:] == -1).all())
