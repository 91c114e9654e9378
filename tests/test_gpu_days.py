"""GPU: the matrix-core kernels of the pattern form (16 days per block), at the
day counts and line lengths where a day group, a tile, a column run or an LDS
stage ends, against the FP64 oracle and against one call per day.

Tolerances: a sum has at most K * degree terms of one sign (demand and ratios
are non-negative), so FP32 products are within 300 * 2^-24 < 2e-5 of each entry
(FP64: 300 * 2^-53 < 4e-14).  A gradient sums residuals of both signs and is
held to its largest entry with the same factor times the residual's
cancellation, below 10 here.  Every day is a matrix-core column of its own, so
one call for n days gives the bits of n calls.
"""
import numpy as np
import pytest

import oracle as orc
import paper_1901_09266_amd as dode
from synth import make_instance, make_perms, chunk_h_blocks
from gpu_helpers import say, make_dar, dev, dequantized_values, rel, rel_elem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DT = {"f64": torch.float64}


def dt_of(storage):
    return DT.get(storage, torch.float32)


def run_all(dar, Q, X):
    n, (P, L, T, H, K) = Q.shape[0], dar.dims
    Xh = torch.empty((n, H, L), dtype=Q.dtype, device="cuda")
    G = torch.empty_like(Q)
    out = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(4)]
    dode.dode_apply(dar, 0, Q, Xh)
    dode.dode_grad(dar, 0, Q, X, G)
    dode.dode_loss(dar, 0, Q, X, out[3])
    dode.dode_metrics(dar, 0, Q, X, loss=out[0], kkt=out[1], r2=out[2])
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in [Xh, G] + out]


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "fp8"])
@pytest.mark.parametrize("P,L,T,H,K,n", [
    (1, 1, 1, 1, 1, 2),          # a single entry
    (5, 7, 4, 6, 3, 3),          # H > T, one short tile each way
    (64, 128, 6, 6, 2, 16),      # whole tiles, a whole group
    (65, 129, 6, 4, 5, 17),      # one line past a tile, one day past a group, H < T, K > H
    (30, 1030, 5, 5, 3, 9),      # more tiles than waves, residual rows a lag at a time
    (1100, 40, 4, 4, 3, 8),      # demand rows a lag at a time, unions of many column runs
    (6, 2600, 3, 3, 2, 5),       # lines too long to stage: one-day kernels
    (4, 1400, 2, 2, 1, 3),       # too long in FP64 only
    # the same edges in passes large enough for the matrix cores (2^22 products)
    (12, 14, 2400, 2402, 3, 70),
    (64, 128, 300, 300, 2, 16),
    (65, 129, 200, 198, 5, 17),
    (30, 1030, 100, 100, 3, 9),
    (1100, 40, 80, 80, 3, 8),
    (4, 1400, 250, 250, 1, 60),
])
def test_days_match_oracle_and_single_days(storage, P, L, T, H, K, n):
    inst = make_instance(P=P, L=L, T=T, H=H, K=K, sizes=(n,), inc=1.0 if P == 1 else 0.06,
                         pattern="bernoulli", demand="gamma", x_dtype="f32", seed=321)
    say("days", storage, P, L, n)
    dt = dt_of(storage)
    rng = np.random.default_rng(7)
    Q = (inst.qstar * rng.uniform(0.5, 1.5, inst.qstar.shape)).astype(np.float32)
    Q[rng.random(Q.shape) < 0.1] = 0.0
    dar = make_dar(inst, storage)
    Qd, Xd = dev(Q, dt), dev(inst.x, dt)
    got = run_all(dar, Qd, Xd)
    one = [run_all(dar, Qd[d:d + 1].contiguous(), Xd[d:d + 1].contiguous()) for d in range(n)]
    for k, a in enumerate(got):
        b = np.concatenate([o[k] for o in one])
        if k < 2:
            assert np.array_equal(a, b)
        else:   # FP64 sums in another order
            np.testing.assert_allclose(a, b, rtol=1e-11, atol=1e-300)
    W = dequantized_values(inst, storage)[0]
    Q64, X64 = Q.astype(np.float64), inst.x.astype(np.float64)
    tol = 4e-14 if storage == "f64" else 2e-5
    for d in (0, n // 2, n - 1):
        assert rel_elem(got[0][d], orc.apply(inst, W, Q64[d]).reshape(H, L)) <= tol
        assert rel(got[1][d], orc.grad(inst, W, Q64[d], X64[d]).reshape(T, P)) <= 10 * tol
        lo = orc.loss(inst, W, Q64[d], X64[d])
        assert abs(got[2][d] - lo) <= 10 * tol * lo


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("sizes", [(3,), (33,), (37, 16, 1)])
def test_plan_minibatches_by_day_groups(storage, sizes):
    """FP64 and FP32 plans step their days in groups: loss history against the
    oracle, and every day the same bits in a plan that groups them otherwise."""
    inst = make_instance(P=37, L=90, T=20, H=22, K=4, sizes=sizes, inc=0.15, pattern="corridor",
                         demand="gamma", x_dtype="f32", seed=323)
    say("plan day groups", storage, sizes)
    E, batch = 3, 5 * inst.L
    perms = make_perms(324, E, inst.C, inst.H)
    dt = dt_of(storage)
    dar = make_dar(inst, storage)
    p = dode.make_params(epochs=E, batch_rows=batch, eta=5.0)

    def solve(days):
        X = dev(inst.x[days], dt)
        Q = torch.zeros((len(days), inst.T, inst.P), dtype=dt, device="cuda")
        A = torch.zeros_like(Q)
        h = dode.spgd_solve(dar, inst.day_cluster[days], X, Q, A, p, perm=perms, loss_hist=True)
        torch.cuda.synchronize()
        return Q.cpu().numpy(), A.cpu().numpy(), h

    Q, A, hist = solve(np.arange(inst.D))
    order = np.arange(inst.D)[::-1].copy()
    for a, b in zip((Q, A, hist), solve(order)):
        assert np.array_equal(a[order], b)
    W = dequantized_values(inst, storage)
    _, _, ho = orc.spgd(inst, inst.x.astype(np.float64), perms, E,
                        chunk_h_blocks(inst.L, inst.H, batch), optimizer=0, eta=5.0, W=W)
    tol = 1e-10 if storage == "f64" else 1e-3
    assert np.max(np.abs(hist - ho) / ho) <= tol


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("T", [16, 40])   # one day per block, 16 days per block
def test_plan_nonfinite_values_stay_on_the_pattern(storage, T):
    """Minibatch steps on infinite demand and counts against the sparse pattern
    kernels (kernel_path 1): the same entries are finite, and equal within the
    rounding of two summation orders over two epochs."""
    inst = make_instance(P=40, L=64, T=T, K=3, sizes=(40,), inc=0.1, pattern="corridor",
                         x_dtype="f64", seed=313)
    say("plan, non-finite", storage)
    dt = dt_of(storage)
    dar = make_dar(inst, storage)
    x, q0 = inst.x.copy(), np.zeros((inst.D, inst.T, inst.P))
    x[3, 5, 10], x[7, 2, 40], q0[11, 4, 20] = np.nan, np.inf, np.inf
    out = []
    for path in (0, 1):
        p = dode.make_params(epochs=2, batch_rows=4 * inst.L, eta=5.0, kernel_path=path,
                             check_finite=0)
        plan = dode.spgd_plan_create(dar, inst.day_cluster, p,
                                     perm=make_perms(314, 2, inst.C, inst.H), stream=0)
        dode.spgd_plan_load(plan, dev(x, dt), dev(q0, dt))
        dode.spgd_run(plan, 0, 2)
        Q = torch.empty((inst.D, inst.T, inst.P), dtype=dt, device="cuda")
        A = torch.empty_like(Q)
        dode.spgd_plan_store(plan, Q, A)
        torch.cuda.synchronize()
        out.append((Q.cpu().numpy(), A.cpu().numpy()))
    for a, b in zip(*out):
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
        m = np.isfinite(b)
        assert m.mean() > 0.9
        assert np.max(np.abs(a[m] - b[m])) <= 20 * (2.3e-14 if storage == "f64" else 1.2e-5) * np.max(np.abs(b[m]))


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("T", [8, 700])   # one day per block, 16 days per block
def test_nonfinite_values_stay_on_the_pattern(storage, T):
    """A NaN or infinite demand or count of one day reaches the entries that
    the pattern connects it to, of that day, and no other."""
    inst = make_instance(P=40, L=64, T=T, K=3, sizes=(9,), inc=0.1, pattern="corridor",
                         x_dtype="f64", seed=325)
    say("days, non-finite", storage)
    dt = dt_of(storage)
    dar = make_dar(inst, storage)
    Q, X = inst.qstar.copy(), inst.x.copy()
    Q[2, 4, 20], Q[5, 1, 3], X[7, 5, 10] = np.inf, np.nan, np.nan
    Qd, Xd = dev(Q, dt), dev(X, dt)
    got = run_all(dar, Qd, Xd)
    for d in range(9):
        one = run_all(dar, Qd[d:d + 1].contiguous(), Xd[d:d + 1].contiguous())
        for a, b in zip(got[:2], one[:2]):
            np.testing.assert_array_equal(a[d], b[0])
    assert np.isfinite(got[0]).mean() > 0.9
