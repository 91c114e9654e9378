"""GPU: ratio calls of few paths, whose days are split over parts (or which take
the two-kernel form), against the oracle: parts that end inside a pattern, a
pattern with fewer day groups than parts, no costs, a scratch limit below one
part's sums.

Bars of the other ratio tests: FP64 1e-12 (the same operations in another
grouping), FP32 2e-5 against the oracle's binary32 walk (sums of n days in FP32
add at most n/2 ulps to the windows' few)."""
import numpy as np
import pytest

import oracle as orc
import paper_1901_09266_amd as dode
from synth import make_speed_instance
from gpu_helpers import say, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f64", [True, False])
@pytest.mark.parametrize("limit", [None, "1000"])
@pytest.mark.parametrize("lens,H,K,sizes,costs", [
    ((1, 7, 20), 24, 6, (200, 3, 77), True),      # 6 parts in FP32; patterns of 1 and 10 groups of 8 days
    ((20, 0, 5), 64, 3, (163,), False),           # the last group of the last part is short
    ((8,), 20, 12, (130, 66), True),              # FP64 in 2 links and 2 days a step
    ((100, 3), 12, 12, (24,), True),              # many segments, few days: two kernels
])
def test_parts_match_oracle(monkeypatch, f64, limit, lens, H, K, sizes, costs):
    if limit:
        monkeypatch.setenv("DODE_DAR_SCRATCH_BYTES", limit)
    say("ratio parts", f64, limit, lens, H, K, sizes)
    rng = np.random.default_rng(51)
    si = make_speed_instance(L=40, P=4, H=H, sizes=sizes, inc=0.1, seed=52)
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    link = rng.integers(0, si.L, ptr[-1]).astype(np.int32)
    t = torch.float64 if f64 else torch.float32
    dptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    out = dode.dode_dar_patterns_from_speeds(
        dev(ptr, torch.int32), dev(link, torch.int32), dev(si.link_len, t), dev(si.speed, t), dptr,
        si.dt, H, K, with_costs=costs)
    torch.cuda.synchronize()
    Rr, cost = out if costs else (out[0] if isinstance(out, tuple) else out, None)
    walk = "f64" if f64 else "f32"
    for q in range(len(sizes)):
        sp = si.speed[dptr[q]:dptr[q + 1]].astype(np.float64)
        Ro = orc.dar_from_speeds(ptr, link, si.link_len, sp, si.dt, H, K, walk=walk)
        assert np.max(np.abs(Rr[q].cpu().numpy() - Ro)) <= (1e-12 if f64 else 2e-5)
        if costs:
            co = orc.path_costs(ptr, link, si.link_len, sp, si.dt, H, walk=walk)
            err = np.abs(cost[q].cpu().numpy() - co) / np.maximum(co, 1.0)
            assert np.max(err) <= (1e-13 if f64 else 2e-7)


@pytest.mark.parametrize("f64", [True, False])
@pytest.mark.parametrize("lens,H,K,sizes", [
    ((1, 7, 20), 24, 6, (200, 3, 77)),            # parts in some patterns of a launch
    ((20, 9), 100, 3, (365, 340, 64, 1, 500)),    # blocks for all patterns, few for one
    ((30, 70), 24, 12, (365, 24, 100)),           # many segments
    ((5,) * 9, 288, 16, (96,) * 18),              # more patterns than a launch
])
def test_pattern_has_the_same_bits_alone(f64, lens, H, K, sizes):
    """In a call of its own, and without costs."""
    say("ratio parts alone", f64, lens, H, K, sizes)
    rng = np.random.default_rng(53)
    n_links = 30
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    link = dev(rng.integers(0, n_links, ptr[-1]), torch.int32)
    t = torch.float64 if f64 else torch.float32
    D = sum(sizes)
    dptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    length, speed = dev(rng.random(n_links) + 0.2, t), dev(rng.random((D, n_links, H)) + 0.3, t)
    paths = dev(ptr, torch.int32), link, length
    Rr, cost = dode.dode_dar_patterns_from_speeds(*paths, speed, dptr, 1440.0 / H, H, K, with_costs=True)
    for q in range(len(sizes)):
        sp = speed[dptr[q]:dptr[q + 1]].contiguous()
        Rq, cq = dode.dode_dar_costs_from_speeds(*paths, sp, 1440.0 / H, H, K)
        Rn = dode.dode_dar_from_speeds(*paths, sp, 1440.0 / H, H, K)
        torch.cuda.synchronize()
        assert torch.equal(Rr[q], Rq) and torch.equal(cost[q], cq) and torch.equal(Rr[q], Rn)
