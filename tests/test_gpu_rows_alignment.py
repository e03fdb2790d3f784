"""GPU: the row form's positions written to an array that starts between 16-byte boundaries (two-byte stores), and to
one that does not, with pair counts around whole groups of eight: the same bits from both."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_13808_amd as dropit
from dropit_inputs import activation
from gpu_util import to_device, to_host

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


@pytest.mark.parametrize("shape", [(40000, 2), (9000, 16), (1000, 777), (300, 4096), (3, 65536), (131072, 1)])
@pytest.mark.parametrize("gamma", [0.0, 0.5, 0.9, 0.999])
def test_sparse_and_full_rows(shape, gamma):
    """One pair per thread (rows with fewer than eight pairs, or few pairs in all) and eight, against the flat indices."""
    print("rows", shape, gamma, flush=True)
    x = activation(shape, "normal", 67 + shape[1], "bf16")
    want_v, want_i = oracle.compress(x, oracle.keep_count(x.size, gamma))
    vals, col, rowptr = dropit.compress_rows(to_device(x), gamma)
    torch.cuda.synchronize()
    assert to_host(vals).tobytes() == want_v.tobytes()
    assert np.array_equal(col.cpu().numpy().view(np.uint16), (want_i % shape[1]).astype(np.uint16))
    assert np.array_equal(rowptr.cpu().numpy(), np.searchsorted(want_i, np.arange(shape[0] + 1, dtype=np.int64) * shape[1]))
