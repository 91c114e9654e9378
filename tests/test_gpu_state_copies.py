"""GPU: the copies between the caller's days and the plan's state, at the day
counts and row lengths where a block, a wave or a vector of four ends, in both
plan layouts: what a plan loads it stores, bit for bit, negative and NaN demand
projected onto zero; and the scan for non-finite counts finds one anywhere."""
import numpy as np
import pytest

import paper_1901_09266_amd as dode
from synth import make_instance
from gpu_helpers import say, make_dar, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("P,T,sizes", [
    (1, 1, (1,)),
    (3, 2, (3, 5)),          # less than a vector; clusters interleaved
    (4, 3, (31,)),
    (5, 3, (32,)),           # a vector and one column; a whole block of days
    (33, 2, (17, 16)),       # one column past a wave's 32; a block and one day
    (127, 2, (4,)),          # every vector in flight, the last one short
    (130, 5, (65,)),         # a second round of vectors
])
def test_plan_stores_what_it_loads(storage, P, T, sizes):
    inst = make_instance(P=P, L=9, T=T, K=1, sizes=sizes, inc=1.0 if P < 8 else 0.3,
                         pattern="bernoulli", x_dtype="f32", seed=421)
    say("state copies", storage, P, T, sizes)
    dt = torch.float64 if storage == "f64" else torch.float32
    rng = np.random.default_rng(422)
    day_cluster = rng.permutation(inst.day_cluster).astype(np.int32)
    Q = rng.normal(size=(inst.D, T, P))
    Q[rng.random(Q.shape) < 0.05] = np.nan
    A = rng.normal(size=Q.shape)
    Qd, Ad = dev(Q, dt), dev(A, dt)
    dar = make_dar(inst, storage)
    p = dode.make_params(epochs=1, batch_rows=9, eta=1.0)
    plan = dode.spgd_plan_create(dar, day_cluster, p)
    X = dev(inst.x, dt)
    dode.spgd_plan_load(plan, X, Qd, Ad)
    Qo, Ao = torch.full_like(Qd, 7.0), torch.full_like(Ad, 7.0)
    dode.spgd_plan_store(plan, Qo, Ao)
    torch.cuda.synchronize()
    assert torch.equal(Qo, torch.where(Qd > 0, Qd, torch.zeros_like(Qd)))
    assert torch.equal(Ao, Ad)
    flat = X.view(-1)
    for i in {0, 1, flat.numel() // 2, flat.numel() - 1} - {flat.numel()}:
        old = flat[i].item()
        flat[i] = float("inf")
        with pytest.raises(dode.DodeError):
            dode.spgd_plan_load(plan, X, Qd, Ad)
        flat[i] = old
    dode.spgd_plan_load(plan, X, Qd, Ad)
