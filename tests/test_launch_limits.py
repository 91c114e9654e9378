"""Launch rules against HIP's limit of 2^32 - 1 threads along a grid's x, without
a GPU: the rules are plain functions of the sizes, called in the library."""
import ctypes
import os

import pytest

from paper_1901_09266_amd import _lib

LIMIT = 2 ** 32 - 1


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(_lib.LIB_PATH):
        from paper_1901_09266_amd.build import build
        build()
    return _lib.lib()


@pytest.mark.parametrize("f64,K,seg", [(False, 6, 8), (False, 9, 4), (True, 6, 4), (True, 16, 2)])
def test_ratio_launches_stay_below_the_limit(L, f64, K, seg):
    fn = L._Z18dar_fused_patternsbiiiii   # (f64, n_paths, longest, H, H_speed, K)
    fn.argtypes = [ctypes.c_bool] + [ctypes.c_int32] * 5
    fn.restype = ctypes.c_int32
    for n_paths in (1, 450, 52_000, 52_500, 262_144, 900_000, 2_000_000):
        for H in (1, 63, 64, 288):
            for longest in (0, 1, seg, seg + 1, 16 * seg):
                n = fn(f64, n_paths, longest, H, H, K)
                threads = n_paths * ((H + 62) // 63) * 64 * max(1, -(-longest // seg))
                assert 0 <= n <= 16 and n * threads <= LIMIT
                assert n == min(16, LIMIT // threads)   # and no smaller than it has to be
            assert fn(f64, n_paths, 16 * seg + 1, H, H, K) == 0   # two kernels
