"""GPU: the one-day forward walk in launches that fill the chip, where sparse
rows (and FP8) take four entries of a lag at a time.  Every form adds a row's
products in the same order, so a day has the same bits in a plan of many days
as alone, in a launch too small for the change of form.  Losses are FP64 sums of
H * L squares that the loss pass of one day may add in another order: two such
sums are within 2 * H * L * 2^-53 of each other."""
import numpy as np
import pytest

import paper_1901_09266_amd as dode
from synth import make_instance, make_perms
from gpu_helpers import say, make_dar, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def solve(dar, inst, days, X, perms, dt):
    p = dode.make_params(epochs=2, batch_rows=inst.H * inst.L, eta=5.0, kernel_path=1)
    plan = dode.spgd_plan_create(dar, np.zeros(len(days), np.int32), p, perm=perms)
    Q = torch.zeros((len(days), inst.T, inst.P), dtype=dt, device="cuda")
    A = torch.zeros_like(Q)
    loss = torch.empty((2, len(days)), dtype=torch.float64, device="cuda")
    dode.spgd_plan_load(plan, X[days].contiguous(), Q, A)
    dode.spgd_run(plan, 0, 2, loss=loss)
    dode.spgd_plan_store(plan, Q, A)
    torch.cuda.synchronize()
    return Q, A, loss


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16", "fp8"])
@pytest.mark.parametrize("P,L,T,H,K,inc,pattern", [
    (28, 83, 24, 24, 3, 0.1, "corridor"),    # links of 2.7 ODs, at most 9; half a block without links
    (9, 289, 22, 24, 2, 0.08, "corridor"),   # links of 0.7 ODs, at most 3: 8-entry form when small
    (26, 64, 24, 23, 4, 0.3, "bernoulli"),   # links of 8 ODs, at most 14: FP8 alone changes form
    (70, 257, 24, 24, 3, 0.02, "bernoulli"), # one link in a block of its own; empty rows
    (26, 128, 24, 24, 3, 0.003, "bernoulli"),  # a link per OD: waves whose links have no entry
])
def test_day_has_the_same_bits_in_a_full_launch(storage, P, L, T, H, K, inc, pattern):
    D = 48   # 24 intervals a minibatch: more than 1024 blocks
    inst = make_instance(P=P, L=L, T=T, H=H, K=K, sizes=(D,), inc=inc, pattern=pattern,
                         demand="gamma", x_dtype="f32", seed=443)
    say("walk forms", storage, P, L, K, inc)
    dt = torch.float64 if storage == "f64" else torch.float32
    dar = make_dar(inst, storage)
    X = dev(inst.x, dt)
    perms = make_perms(442, 2, 1, H)
    Q, A, loss = solve(dar, inst, list(range(D)), X, perms, dt)
    assert torch.isfinite(Q).all() and (Q > 0).any()
    for d in (0, 17, D - 1):
        q, a, l = solve(dar, inst, [d], X, perms, dt)
        assert torch.equal(Q[d], q[0]) and torch.equal(A[d], a[0])
        assert torch.all((loss[:, d] - l[:, 0]).abs() <= 2.0 ** -52 * H * L * l[:, 0])
