"""GPU: a handle carries the packed values of the 16-day kernels only where those
can run: rows of 16 days that a block cannot stage leave the two sliced copies."""
import numpy as np
import pytest

import paper_1901_09266_amd as dode
from gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,L,storage,packed", [
    (64, 1500, "f64", False),    # 16 FP64 days of 1500 links: 188 KB
    (1500, 64, "f64", False),
    (64, 1216, "f64", True),     # 152 KB
    (64, 1500, "f32", True),
    (64, 2500, "f32", False),
])
def test_no_packed_values_for_rows_that_cannot_be_staged(P, L, storage, packed):
    K, T = 2, 40
    say("handle memory", P, L, storage)
    dar = dode.dar_create(P, L, T, T, K, np.arange(L + 1, dtype=np.int32) * P,
                          np.tile(np.arange(P, dtype=np.int32), L), np.full((1, K, T, P * L), 0.5),
                          storage=storage)
    esz = 8 if storage == "f64" else 4
    slices = K * T * esz * (-(-L // 64) * 64 * P + -(-P // 64) * 64 * L)
    index = 16 * 4 * P * L   # at most 16 index arrays of an entry each
    info = dode.dar_info(dar)
    assert slices <= info["device_bytes"]
    assert (info["device_bytes"] > slices + index) == packed
    Q = torch.ones((33, T, P), dtype=torch.float64 if storage == "f64" else torch.float32, device="cuda")
    X = torch.empty((33, T, L), dtype=Q.dtype, device="cuda")
    dode.dode_apply(dar, 0, Q, X)
    torch.cuda.synchronize()
    want = torch.full_like(X, P * K * 0.5)   # exact in FP32
    want[:, 0] = P * 0.5
    assert torch.equal(X, want)
