"""GPU: the matrix-core forward product with the demand shared by a block, at the
sizes where its blocks, phases and groups end.

Its products come in the order of the one-launch kernels (kernel_path 2), so the
solves are the same bits, for every width of the day groups; refinement steps
(which path 2 runs through the same launches) are compared between widths."""
import numpy as np
import pytest

import paper_1901_09266_amd as dode
from synth import make_instance, make_perms
from gpu_helpers import say, make_dar, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def solve(inst, dar, perms, **kw):
    rows = 3 if inst.H < 50 else 60
    p = dode.make_params(epochs=2, batch_rows=rows * inst.L, eta=5.0, **kw)
    plan = dode.spgd_plan_create(dar, inst.day_cluster, p, perm=perms)
    Q = torch.zeros((inst.D, inst.T, inst.P), dtype=torch.float32, device="cuda")
    A = torch.zeros_like(Q)
    dode.spgd_plan_load(plan, dev(inst.x, torch.float32), Q, A)
    dode.spgd_run(plan, 0, 2)
    dode.spgd_plan_store(plan, Q, A)
    torch.cuda.synchronize()
    return Q, A


@pytest.mark.parametrize("storage,refine", [("bf16", 0), ("fp8", 0), ("fp8", 1)])
@pytest.mark.parametrize("P,L,T,H,K,sizes,inc,pattern", [
    (3, 5, 4, 6, 2, (3,), 1.0, "bernoulli"),             # one tile; H > T
    (40, 129, 9, 9, 3, (33, 4), 0.1, "corridor"),        # a second block of one tile; a group of one day
    (150, 264, 12, 10, 12, (17,), 0.08, "corridor"),     # several phases of lags; H < T
    (260, 300, 6, 6, 3, (20,), 0.05, "bernoulli"),       # every OD in a block; one lag per phase at 64 days
    (600, 70, 5, 5, 3, (9,), 0.05, "bernoulli"),         # one lag fits at 16 days only
    (1100, 40, 4, 4, 2, (5,), 0.05, "bernoulli"),        # too long: one wave per tile group
    # launches large enough that bf16 and corrected values share the demand too
    (40, 129, 200, 200, 3, (33, 130), 0.1, "corridor"),
    (150, 264, 120, 118, 12, (170,), 0.08, "corridor"),
    (260, 300, 100, 100, 3, (400,), 0.05, "bernoulli"),
])
def test_forward_blocks_give_the_one_launch_bits(storage, refine, P, L, T, H, K, sizes, inc, pattern):
    inst = make_instance(P=P, L=L, T=T, H=H, K=K, sizes=sizes, inc=inc, pattern=pattern,
                         demand="gamma", x_dtype="f32", seed=431)
    say("forward blocks", storage, refine, P, L, K, sizes)
    perms = make_perms(432, 2, inst.C, inst.H)
    dar = make_dar(inst, storage, correction=True) if refine else make_dar(inst, storage)
    base = solve(inst, dar, perms, day_tile=16, kernel_path=2, refine_steps=refine)
    assert torch.isfinite(base[0]).all() and (base[0] > 0).any()
    for tile in (16, 32, 64):
        got = solve(inst, dar, perms, day_tile=tile, kernel_path=0, refine_steps=refine)
        for a, b in zip(base, got):
            assert torch.equal(a, b), tile
