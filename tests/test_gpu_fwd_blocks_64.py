"""GPU: the bfloat16 forward product with the demand shared by a block, in groups of
64 days and launches large enough to use it (from 3072 waves: minibatches of 60
rows, the clusters' groups of 64 days, two tiles of 16 links a wave).  The bits are those of
the one-launch kernels (kernel_path 2) in groups of 16 days."""
import pytest

from synth import make_instance, make_perms
from gpu_helpers import say, make_dar
from test_gpu_fwd_blocks import solve

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,L,T,H,K,sizes,inc,pattern", [
    (40, 129, 60, 60, 3, (33, 385), 0.1, "corridor"),     # two lags per phase; 3840 waves, a group of one day
    (150, 264, 62, 60, 12, (257,), 0.08, "corridor"),     # one lag per phase; 3600 waves, a last group of one day; H < T
    (250, 300, 60, 61, 3, (270,), 0.05, "bernoulli"),     # every OD in a block, 65,536 bytes a lag, the most; H > T
])
def test_wide_forward_blocks_give_the_one_launch_bits(P, L, T, H, K, sizes, inc, pattern):
    inst = make_instance(P=P, L=L, T=T, H=H, K=K, sizes=sizes, inc=inc, pattern=pattern,
                         demand="gamma", x_dtype="f32", seed=433)
    say("wide forward blocks", P, L, K, sizes)
    perms = make_perms(434, 2, inst.C, inst.H)
    dar = make_dar(inst, "bf16")
    base = solve(inst, dar, perms, day_tile=16, kernel_path=2)
    assert torch.isfinite(base[0]).all() and (base[0] > 0).any()
    got = solve(inst, dar, perms, day_tile=64, kernel_path=0)
    for a, b in zip(base, got):
        assert torch.equal(a, b)
