"""GPU: the one-kernel ratio construction at the sizes where a segment of links,
a group of days, a run of 63 intervals or a launch of 16 patterns ends, and the
two-kernel form that longer paths take, against the FP64 oracle.

FP64 bars as in the other ratio tests (1e-12: the same operations in another
grouping); FP32 against the oracle's binary32 walk, 2e-5 on windows of about
one interval (end points within a few ulps of the path's travel time)."""
import numpy as np
import pytest

import oracle as orc
import paper_1901_09266_amd as dode
from synth import make_speed_instance
from gpu_helpers import say, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def ragged(lens, L, rng):
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    link = np.concatenate([rng.permutation(L)[:m] if m <= L else rng.integers(0, L, m)
                           for m in lens] + [np.zeros(0, int)]).astype(np.int32)
    return ptr, link


@pytest.mark.parametrize("f64", [True, False])
@pytest.mark.parametrize("lens,H,K,sizes", [
    ((1, 7, 8, 9, 0, 17), 63, 6, (8,)),            # a path without links, one interval run
    ((3, 4, 5, 16, 2), 64, 3, (9, 1)),             # one interval past the run, day groups of 1 and 8+1
    ((8, 15, 31), 12, 8, (2,) * 18),               # more patterns than a launch takes
    ((2, 64, 33, 5), 20, 16, (5,)),                # all 16 lags; FP64 past its 32 links: two kernels
    ((127, 128, 1), 24, 6, (3,)),                  # the longest path of one block in FP32
    ((129, 4), 24, 6, (3, 2)),                     # one link more: two kernels
])
def test_segments_match_oracle(f64, lens, H, K, sizes):
    rng = np.random.default_rng(41)
    si = make_speed_instance(L=40, P=4, H=H, sizes=sizes, inc=0.1, seed=42)
    ptr, link = ragged(lens, si.L, rng)
    say("ratio segments", f64, lens, H, K, sizes)
    t = torch.float64 if f64 else torch.float32
    dptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    Rr, cost = dode.dode_dar_patterns_from_speeds(
        dev(ptr, torch.int32), dev(link, torch.int32), dev(si.link_len, t), dev(si.speed, t), dptr,
        si.dt, H, K, with_costs=True)
    torch.cuda.synchronize()
    Rr, cost = Rr.cpu().numpy(), cost.cpu().numpy()
    walk = "f64" if f64 else "f32"
    for q in range(len(sizes)):
        sp = si.speed[dptr[q]:dptr[q + 1]].astype(np.float64)
        Ro = orc.dar_from_speeds(ptr, link, si.link_len, sp, si.dt, H, K, walk=walk)
        co = orc.path_costs(ptr, link, si.link_len, sp, si.dt, H, walk=walk)
        assert np.max(np.abs(Rr[q] - Ro)) <= (1e-12 if f64 else 2e-5)
        assert np.max(np.abs(cost[q] - co) / np.maximum(co, 1.0)) <= (1e-13 if f64 else 2e-7)
