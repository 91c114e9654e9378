"""GPU: the loss gradient with respect to the assignment values with the day rows
staged in LDS, at the counts where its days, entries and lags end, and with rows
too long to stage.  Each value is an FP64 sum over the days of exact products of
the stored residuals and demand, rounded once: FP64 within n_days * 2^-53 of the
sum of magnitudes, FP32 within its own rounding, 2^-24, of the value."""
import numpy as np
import pytest

import paper_1901_09266_amd as dode
from synth import make_instance
from gpu_helpers import say, make_dar, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("P,L,T,H,K,n,inc", [
    (1, 1, 2, 2, 1, 1, 1.0),
    (7, 40, 4, 5, 3, 8, 0.3),        # a whole stage of days; H > T
    (30, 103, 5, 4, 3, 9, 1.0),      # 3090 entries: a second block; H < T
    (20, 60, 3, 3, 2, 17, 0.2),      # two stages and a day
    (500, 700, 2, 2, 2, 3, 0.02),    # staged in FP32, too long in FP64
    (900, 1200, 2, 2, 2, 3, 0.01),   # too long in both
])
def test_value_gradient(storage, P, L, T, H, K, n, inc):
    inst = make_instance(P=P, L=L, T=T, H=H, K=K, sizes=(n,), inc=inc, pattern="bernoulli",
                         demand="gamma", x_dtype="f32", seed=441)
    say("value gradient", storage, P, L, n)
    dt = torch.float64 if storage == "f64" else torch.float32
    dar = make_dar(inst, storage)
    Q, X = dev(inst.qstar * 0.7, dt), dev(inst.x, dt)
    Xh = torch.empty((n, H, L), dtype=dt, device="cuda")
    dode.dode_apply(dar, 0, Q, Xh)
    dW = torch.empty((K, T, len(inst.col_idx)), dtype=dt, device="cuda")
    dode.dode_loss_bwd(dar, 0, Q, X, 1.0, dW=dW)
    torch.cuda.synchronize()
    R, q = (Xh - X).double().cpu().numpy(), Q.double().cpu().numpy()
    a = np.repeat(np.arange(L), np.diff(inst.row_ptr))
    p = np.asarray(inst.col_idx)
    got = dW.double().cpu().numpy()
    for l in range(K):
        for t in range(T):
            if t + l >= H:
                assert not got[l, t].any()
                continue
            terms = 2.0 * R[:, t + l, a] * q[:, t, p]
            want, size = terms.sum(0), np.abs(terms).sum(0)
            tol = (n + 2) * 2.0 ** -53 * size + (2.0 ** -24 * np.abs(want) if storage == "f32" else 0)
            assert np.all(np.abs(got[l, t] - want) <= tol)
