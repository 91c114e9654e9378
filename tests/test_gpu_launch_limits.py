"""GPU: calls whose work, in one launch, would pass HIP's limit of 2^32 - 1
threads along a grid's x."""
import numpy as np
import pytest

import paper_1901_09266_amd as dode
from gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_ratios_of_more_patterns_than_a_launch_can_take():
    """262 200 paths, one of 128 links (blocks of 1024 threads), 16 patterns of
    one day: 15 patterns fill a launch.  Each pattern alone gives the same bits."""
    n_paths, L, H, C = 262_200, 130, 63, 16
    say("ratio launch limit", n_paths, C)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    deg = torch.ones(n_paths, dtype=torch.int64, device="cuda")
    deg[7] = 128
    ptr = torch.zeros(n_paths + 1, dtype=torch.int32, device="cuda")
    ptr[1:] = deg.cumsum(0)
    link = torch.randint(0, L, (int(ptr[-1]),), generator=g, device="cuda", dtype=torch.int32)
    length = torch.rand(L, generator=g, device="cuda") + 0.5
    speed = torch.rand((C, L, H), generator=g, device="cuda") + 0.5
    Rr, cost = dode.dode_dar_patterns_from_speeds(ptr, link, length, speed,
                                                  np.arange(C + 1, dtype=np.int32), 5.0, H, 1,
                                                  with_costs=True)
    for q in (0, 7, 14, 15):
        Rq, cq = dode.dode_dar_costs_from_speeds(ptr, link, length, speed[q:q + 1], 5.0, H, 1)
        torch.cuda.synchronize()
        assert torch.equal(Rr[q], Rq) and torch.equal(cost[q], cq)
        assert (cost[q] > 0).all() and (Rr[q] >= 0).all()


def test_state_copies_of_more_days_and_rows_than_a_launch_can_take():
    """65,535 days of 8,200 intervals (blocks of 32 days of one row, 256 threads):
    loaded into a plan and stored back, the demand is the same."""
    D, T, P, L = 65_535, 8_200, 1, 2
    say("copy launch limit", D, T)
    dar = dode.dar_create(P, L, T, T, 1, np.array([0, 1, 1], np.int32), np.zeros(1, np.int32),
                          np.ones((1, 1, T, 1)), storage="f32")
    p = dode.make_params(epochs=1, batch_rows=T * L, kernel_path=1)
    plan = dode.spgd_plan_create(dar, np.zeros(D, np.int32), p, seed=1)
    X = torch.zeros((D, T, L), device="cuda")
    Q = torch.arange(D * T, device="cuda", dtype=torch.float32).reshape(D, T, P)
    out = torch.empty_like(Q)
    dode.spgd_plan_load(plan, X, Q)
    dode.spgd_plan_store(plan, out)
    torch.cuda.synchronize()
    assert torch.equal(out, Q)


def test_handle_of_more_blocks_than_a_launch_can_take():
    """Two lags of 4.2 M intervals: 8.4 M blocks of 512 threads install the values."""
    T, K = 4_200_000, 2
    say("install launch limit", T, K)
    W = np.ones((1, K, T, 1))
    W[0, 1] = 2.0
    dar = dode.dar_create(1, 1, T, T, K, np.array([0, 1], np.int32), np.zeros(1, np.int32), W,
                          storage="bf16")
    Q = torch.arange(T, device="cuda", dtype=torch.float32).remainder(1024).reshape(1, T, 1)
    X = torch.empty_like(Q)
    dode.dode_apply(dar, 0, Q, X)
    torch.cuda.synchronize()
    assert torch.equal(X[0, 0], Q[0, 0]) and torch.equal(X[0, 1:], Q[0, 1:] + 2 * Q[0, :-1])
