"""GPU: the one-day pattern kernels (kernel_path 1) at the degrees where their
walks change form, against the FP64 oracle: rows of up to 8, up to 16 and more
entries, columns that end inside and on a step of 8, more lags in a minibatch
than the residual rows a wave stages, demand rows too long to stage.

Losses after the first epoch carry the rounding of the solve: FP64 1e-10; FP32
values and sums 1e-3, the bounds of the other solves against the oracle."""
import numpy as np
import pytest

import oracle as orc
import paper_1901_09266_amd as dode
from synth import make_instance, make_perms, chunk_h_blocks
from gpu_helpers import say, make_dar, dev, rel, dequantized_values

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "fp8"])
@pytest.mark.parametrize("P,L,T,H,K,inc,hb", [
    (1, 1, 3, 3, 1, 1.0, 2),         # one entry
    (16, 8, 6, 8, 3, 1.0, 3),        # rows of 16, columns of 8 entries
    (17, 9, 6, 4, 3, 1.0, 2),        # rows of 17, columns of 9; H < T
    (8, 64, 5, 5, 2, 1.0, 5),        # rows of 8, columns of 64; whole epoch in one minibatch
    (64, 65, 9, 9, 6, 0.2, 4),       # a second slice of one link
    (65, 256, 9, 10, 4, 0.1, 9),     # a second slice of one OD
    (40, 257, 12, 12, 12, 0.1, 12),  # every lag in the minibatch: more rows than are staged
    (20, 1100, 4, 4, 3, 0.3, 2),     # long residual rows, one or two staged
    (900, 30, 5, 5, 6, 0.05, 2),     # demand of 6 lags staged in FP32, too long in FP64
    (1500, 12, 4, 4, 6, 0.05, 2),    # too long in both
])
def test_pattern_walks_match_oracle(storage, P, L, T, H, K, inc, hb):
    inst = make_instance(P=P, L=L, T=T, H=H, K=K, sizes=(1, 2), inc=inc, pattern="bernoulli",
                         demand="gamma", x_dtype="f32", seed=411)
    say("pattern walks", storage, P, L, K, hb)
    E = 3
    perms = make_perms(412, E, inst.C, inst.H)
    bh = chunk_h_blocks(inst.L, inst.H, hb * L)
    W = dequantized_values(inst, storage)
    dt = torch.float64 if storage == "f64" else torch.float32
    dar = make_dar(inst, storage)
    x64 = inst.x.astype(np.float64)
    Qo, Ao, ho = orc.spgd(inst, x64, perms, E, bh, optimizer=0, eta=5.0, W=W)
    Q = torch.zeros((inst.D, T, P), dtype=dt, device="cuda")
    A = torch.zeros_like(Q)
    p = dode.make_params(epochs=E, batch_rows=hb * L, eta=5.0, kernel_path=1)
    h = dode.spgd_solve(dar, inst.day_cluster, dev(x64, dt), Q, A, p, perm=perms, loss_hist=True)
    torch.cuda.synchronize()
    tol = 1e-10 if storage == "f64" else 1e-3
    assert np.max(np.abs(h - ho) / np.maximum(ho, 1e-12 * np.max(ho))) <= tol
    if storage == "f64":
        assert rel(Q.cpu().numpy(), Qo) <= 1e-8 and rel(A.cpu().numpy(), Ao) <= 1e-8
