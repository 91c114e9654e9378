"""GPU: calls with enough days that the 16-day kernels are the faster form: day
groups and tiles at their edges, minibatch steps, non-finite values. Days are
compared with calls of one day each, where a single day is left to the one-day
kernels, bit for bit (products and sums run in one order in both).

Against the oracle: sums of K * degree terms of one sign within 300 * 2^-24 < 2e-5
(FP64 300 * 2^-53 < 4e-14), gradients ten times that of their largest entry."""
import numpy as np
import pytest

import oracle as orc
import paper_1901_09266_amd as dode
from synth import make_instance, make_perms, chunk_h_blocks
from gpu_helpers import say, make_dar, dev, dequantized_values, rel, rel_elem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def passes(dar, Q, X):
    n, (P, L, T, H, K) = Q.shape[0], dar.dims
    Xh = torch.empty((n, H, L), dtype=Q.dtype, device="cuda")
    G, dQ = torch.empty_like(Q), torch.empty_like(Q)
    loss = torch.empty(n, dtype=torch.float64, device="cuda")
    dode.dode_apply(dar, 0, Q, Xh)
    dode.dode_grad(dar, 0, Q, X, G)
    dode.dode_loss(dar, 0, Q, X, loss)
    dode.dode_loss_bwd(dar, 0, Q, X, 0.75, dQ=dQ)
    torch.cuda.synchronize()
    return Xh, G, dQ, loss


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "fp8"])
@pytest.mark.parametrize("P,L,T,H,K,n", [
    (64, 128, 120, 120, 2, 96),      # whole tiles, whole groups
    (65, 129, 100, 98, 5, 81),       # one line past a tile, one day past a group, H < T
    (30, 1030, 60, 60, 3, 79),       # more tiles than waves, residual rows a lag at a time
    (700, 40, 40, 42, 3, 76),        # demand rows a lag at a time, unions of many column runs; H > T
    (12, 14, 600, 600, 3, 250),      # one tile each way
])
def test_passes_of_many_days(storage, P, L, T, H, K, n):
    inst = make_instance(P=P, L=L, T=T, H=H, K=K, sizes=(n,), inc=0.2, pattern="corridor",
                         demand="gamma", x_dtype="f32", seed=331)
    say("day forms", storage, P, L, n)
    dt = torch.float64 if storage == "f64" else torch.float32
    rng = np.random.default_rng(8)
    Q = (inst.qstar * rng.uniform(0.5, 1.5, inst.qstar.shape)).astype(np.float32)
    Q[rng.random(Q.shape) < 0.1] = 0.0
    dar = make_dar(inst, storage)
    Qd, Xd = dev(Q, dt), dev(inst.x, dt)
    got = passes(dar, Qd, Xd)
    W = dequantized_values(inst, storage)[0]
    tol = 4e-14 if storage == "f64" else 2e-5
    for d in (0, 15, 16, n // 2, n - 1):
        one = passes(dar, Qd[d:d + 1].contiguous(), Xd[d:d + 1].contiguous())
        for a, b in zip(got[:3], one[:3]):
            assert torch.equal(a[d], b[0])
        assert abs(float(got[3][d] - one[3][0])) <= 1e-11 * float(one[3][0])   # FP64 sums in another order
        q64, x64 = Q[d].astype(np.float64), inst.x[d].astype(np.float64)
        assert rel_elem(got[0][d].cpu().numpy(), orc.apply(inst, W, q64).reshape(H, L)) <= tol
        assert rel(got[1][d].cpu().numpy(), orc.grad(inst, W, q64, x64).reshape(T, P)) <= 10 * tol


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("sizes", [(96,), (65, 33, 2)])
def test_minibatches_of_many_days(storage, sizes):
    """Steps and losses in day groups: the days in another order (other groups)
    and single days alone give the same bits; losses against the oracle."""
    inst = make_instance(P=72, L=96, T=40, H=42, K=4, sizes=sizes, inc=0.25, pattern="corridor",
                         demand="gamma", x_dtype="f32", seed=333)
    say("day forms, minibatches", storage, sizes)
    E, batch = 2, 14 * inst.L
    perms = make_perms(334, E, inst.C, inst.H)
    dt = torch.float64 if storage == "f64" else torch.float32
    dar = make_dar(inst, storage)
    p = dode.make_params(epochs=E, batch_rows=batch, eta=5.0)

    def solve(days):
        Q = torch.zeros((len(days), inst.T, inst.P), dtype=dt, device="cuda")
        A = torch.zeros_like(Q)
        h = dode.spgd_solve(dar, inst.day_cluster[days], dev(inst.x[days], dt), Q, A, p, perm=perms,
                            loss_hist=True)
        torch.cuda.synchronize()
        return Q.cpu().numpy(), A.cpu().numpy(), h

    Q, A, hist = solve(np.arange(inst.D))
    order = np.arange(inst.D)[::-1].copy()
    for a, b in zip((Q, A, hist), solve(order)):
        assert np.array_equal(a[order], b)
    for d in (0, 40, inst.D - 1):
        q, a, h = solve(np.array([d]))
        assert np.array_equal(Q[d], q[0]) and np.array_equal(A[d], a[0])
        np.testing.assert_allclose(hist[d], h[0], rtol=1e-11)
    _, _, ho = orc.spgd(inst, inst.x.astype(np.float64), perms, E,
                        chunk_h_blocks(inst.L, inst.H, batch), optimizer=0, eta=5.0,
                        W=dequantized_values(inst, storage))
    assert np.max(np.abs(hist - ho) / ho) <= (1e-10 if storage == "f64" else 1e-3)


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
def test_nonfinite_values_of_many_days(storage):
    """A NaN or infinite demand or count of one day reaches what the pattern
    connects it to, of that day, in passes and in minibatch steps."""
    inst = make_instance(P=72, L=96, T=60, K=3, sizes=(96,), inc=0.25, pattern="corridor",
                         x_dtype="f64", seed=335)
    say("day forms, non-finite", storage)
    dt = torch.float64 if storage == "f64" else torch.float32
    dar = make_dar(inst, storage)
    Q, X = inst.qstar.copy(), inst.x.copy()
    Q[2, 4, 20], Q[50, 1, 3], X[95, 5, 10] = np.inf, np.nan, np.nan
    Qd, Xd = dev(Q, dt), dev(X, dt)
    got = passes(dar, Qd, Xd)
    bad = 0
    for d in (1, 2, 3, 49, 50, 94, 95):
        one = passes(dar, Qd[d:d + 1].contiguous(), Xd[d:d + 1].contiguous())
        for a, b in zip(got[:3], one[:3]):
            np.testing.assert_array_equal(a[d].cpu().numpy(), b[0].cpu().numpy())
            bad += int((~torch.isfinite(a[d])).sum())
    assert 0 < bad < 0.2 * 7 * got[1][0].numel()
    if storage == "bf16":   # steps of 16-day groups are for FP32 and FP64
        return
    p = dode.make_params(epochs=1, batch_rows=20 * inst.L, eta=5.0, check_finite=0)
    perm = make_perms(336, 1, 1, inst.H)

    def solve(days):
        q, a = Qd[days].contiguous(), torch.zeros_like(Qd[days])
        dode.spgd_solve(dar, inst.day_cluster[days], Xd[days].contiguous(), q, a, p, perm=perm)
        torch.cuda.synchronize()
        return q.cpu().numpy(), a.cpu().numpy()

    q, a = solve(list(range(inst.D)))
    assert not np.isfinite(a).all()
    for d in (2, 50, 95):
        for x, y in zip((q, a), solve([d])):
            np.testing.assert_array_equal(x[d], y[0])
