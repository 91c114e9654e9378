"""GPU: the dense solve's residuals carried from the loss of one epoch to the
single minibatch of the next, its loss squares summed for several epochs at a
time, and the column sums with and without the slice's rows in LDS, at the
counts where each of them ends.

With a loss history and without, the iterates are the same bits: both use the
same residual of every row.  The losses are within the FP32 dot products'
rounding (n terms of one sign: n * 2^-24 of the row's value, doubled by the
square), FP64 within 1e-12."""
import numpy as np
import pytest

import oracle as orc
import paper_1901_09266_amd as dode
from gpu_helpers import say, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64, torch.bfloat16])
@pytest.mark.parametrize("m,n,chunk,E", [
    (128, 512, 8192, 3),        # one slice, whole rounds of rows in flight
    (129, 2052, 129, 3),        # a second slice of one row
    (157, 4104, 64, 2),         # several minibatches; rows left after a round
    (8200, 4104, 8200, 2),      # more than 512 blocks: rows read by each wave
    (2100000, 4, 3000000, 4),   # more rows than two epochs' residuals of the scratch
])
def test_epochs_with_and_without_loss(dtype, m, n, chunk, E):
    say("dense epochs", dtype, m, n, chunk)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    t = torch.float64 if dtype == torch.float64 else torch.float32
    B = torch.rand((m, n), generator=g, device="cuda", dtype=torch.float64).to(dtype)
    y = (B.double() @ torch.rand(n, generator=g, device="cuda", dtype=torch.float64)).to(t)
    perms = torch.stack([torch.randperm(m, generator=g, device="cuda") for _ in range(E)]).int()
    out = []
    for loss in (True, False):
        q = torch.zeros(n, dtype=t, device="cuda")
        A = torch.zeros_like(q)
        h = dode.dense_spgd_run(B, y, q, A, perms, chunk, 0.1, loss_hist=loss)
        torch.cuda.synchronize()
        out.append((q, A, h))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    if m > 10000:   # each epoch's loss from a run that ends there
        for e in range(1, E + 1):
            q = torch.zeros(n, dtype=t, device="cuda")
            A = torch.zeros_like(q)
            h = dode.dense_spgd_run(B, y, q, A, perms[:e].contiguous(), chunk, 0.1, loss_hist=True)
            assert np.array_equal(h, out[0][2][:e])
        return
    qo, Ao, ho = orc.dense_spgd(B.double().cpu().numpy(), y.double().cpu().numpy(),
                                perms.cpu().numpy(), chunk, 0.1)
    y2 = float((y.double() ** 2).sum())
    tol = 1e-12 if dtype == torch.float64 else 2 * n * 2.0 ** -24
    assert np.max(np.abs(out[0][2] - ho)) <= tol * y2
