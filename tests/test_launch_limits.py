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


@pytest.mark.parametrize("rows,waves", [(True, 8), (False, 16)])
def test_launches_of_day_groups_stay_below_the_limit(L, rows, waves):
    fn = L._Z15day_launch_fitsilib   # (n_rows, groups, n_tiles, rows)
    fn.argtypes = [ctypes.c_int32, ctypes.c_int64, ctypes.c_int32, ctypes.c_bool]
    fn.restype = ctypes.c_bool
    for n_rows in (1, 7, 288, 1441, 65535):
        for n_tiles in (1, 2, waves - 1, waves, waves + 1, 100):
            threads = 64 * min(n_tiles, waves)
            most = LIMIT // threads // 8 * 8 // n_rows   # grids are multiples of 8 blocks
            for groups in (1, most - 1, most, most + 1, 2 * most, 2 ** 28):
                if groups < 1:
                    continue
                blocks = (n_rows * groups + 7) // 8 * 8
                assert fn(n_rows, groups, n_tiles, rows) == (blocks * threads <= LIMIT)
