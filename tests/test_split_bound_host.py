"""The workspace for K-split partial tiles is sized by the most that a context can need (host
arithmetic, no GPU): no launch of it may use more."""
import ctypes

import pytest

import paper_2510_19470_amd as moe


@pytest.mark.parametrize("n_cu", [256, 304, 8])
@pytest.mark.parametrize("kt_max", [2, 14, 16, 18, 32, 64, 128, 448])
def test_no_launch_uses_more_partial_tiles_than_the_bound(n_cu, kt_max):
    rule = moe.load_library().moe_internal_split_tiles
    used, most = ctypes.c_int32(), ctypes.c_int64()
    for tiles_max in (1, 2, 3, 7, 8, 31, 32, 33, 100, 255, 256, 257, 700):
        peak = 0
        for tiles in range(tiles_max + 1):
            for kt in {2, kt_max // 4 * 2, kt_max}:      # down (one segment) and dX (two) of a context
                if kt < 2:
                    continue
                rule(tiles, ctypes.c_int64(tiles_max), n_cu, kt, ctypes.byref(used), ctypes.byref(most))
                peak = max(peak, used.value)
        rule(tiles_max, ctypes.c_int64(tiles_max), n_cu, kt_max, ctypes.byref(used), ctypes.byref(most))
        assert peak <= most.value <= n_cu
        assert (most.value == 0) == (kt_max < 16)         # fewer than eight pairs of k-steps: never cut
