"""When the expert FFN takes 128-row tiles, and the workspace of their cut contractions (host arithmetic,
no GPU).  The host does not know how the tokens fall: the rule goes by an even routing, but not where
another routing can bring many more tiles."""
import ctypes

import pytest

import paper_2510_19470_amd as moe

N_CU = 256


def tile128(T, d, f, E, k, n_res, gated, backward):
    return bool(moe.load_library().moe_internal_ffn_tile128(T, d, f, E, k, n_res, int(gated), int(backward), N_CU))


@pytest.mark.parametrize("T,d,f,E,k,n_res,gated,backward,want", [
    # measured faster with the smaller tiles, evenly and where all tokens agree (but for 4 % of the first)
    (1999, 1160, 2888, 16, 2, 6, True, False, True), (1999, 1160, 2888, 16, 2, 6, True, True, True),
    (1024, 1024, 4096, 32, 2, 8, False, False, True), (1024, 1024, 4096, 32, 2, 8, False, True, True),
    (200, 2048, 1408, 64, 6, 12, True, False, True), (2000, 768, 1024, 16, 4, 6, True, True, True),
    (751, 664, 384, 64, 3, 11, True, False, True), (64, 4096, 14336, 8, 2, 8, True, False, True),
    (128, 4096, 14336, 8, 2, 8, True, False, True),
    # measured slower, evenly or where the tokens agree
    (4096, 1024, 4096, 16, 2, 6, True, False, False), (4096, 1024, 4096, 16, 2, 6, True, True, False),
    (8192, 2048, 2048, 32, 4, 6, True, False, False), (2034, 768, 2560, 16, 3, 11, True, False, False),
    (6517, 768, 1024, 32, 6, 19, False, False, False), (7216, 1280, 768, 8, 3, 4, False, False, False),
    (128, 4096, 14336, 8, 2, 8, True, True, False), (4096, 2048, 1408, 64, 6, 12, True, True, False),
    (16384, 2048, 1408, 64, 6, 12, True, False, False), (8192, 4096, 14336, 8, 2, 8, True, False, False),
    (100, 64, 64, 8, 2, 0, True, False, False)])
def test_rule_follows_what_was_measured(T, d, f, E, k, n_res, gated, backward, want):
    assert tile128(T, d, f, E, k, n_res, gated, backward) == want


def test_no_routing_brings_more_than_two_rounds_of_larger_tiles():
    for d in (8, 512, 2048, 4096):
        for f in (8, 768, 4096, 14336):
            for E, k in ((4, 1), (8, 2), (64, 6), (256, 16)):
                for n_res in (1, E // 2, E):
                    for T in (129, 200, 1000, 4096, 16384, 200000):
                        for gated in (True, False):
                            if tile128(T, d, f, E, k, n_res, gated, False):
                                cols = -(-f // (128 if gated else 256))
                                assert (T * min(k, n_res) // 256 + n_res) * cols <= 2 * N_CU


@pytest.mark.parametrize("slots", [16, 512, 608])
def test_parts_fit_the_resident_blocks_and_the_workspace(slots):
    parts = moe.load_library().moe_internal_tile128_parts
    for kt in (1, 7, 8, 9, 16, 63, 64, 448):
        most = parts(1, 8, kt)                  # what the workspace is sized with
        assert (most == 1) == (kt < 8)
        for tiles in list(range(0, 70)) + [127, 128, 255, 256, 257, 512, 5000]:
            n = parts(tiles, slots, kt)
            assert 1 <= n <= most and (n == 1 or (tiles * n <= slots and kt // n >= 4))


def tile_us(experts, rows, d, f, gated, backward):
    us = (ctypes.c_double * 2)()
    moe.load_library().moe_internal_ffn_tile_us(experts, rows, d, f, int(gated), int(backward), N_CU, us)
    return us[0], us[1]


@pytest.mark.parametrize("gated,backward", [(True, False), (False, False), (False, True)])
def test_estimate_cuts_contractions_as_the_larger_tiles_do(gated, backward):
    """An odd number of k-steps is rounded up to an even one before the contraction is cut: a launch of 23
    steps has the parts of one of 24.  (dX of the gated expert contracts over two segments: always even.)"""
    for f in (1464, 1208, 952, 568):                # 23, 19, 15 and 9 steps; one more for 56 columns more
        for experts, rows in ((5, 703), (1, 200), (3, 1000), (2, 5000)):
            for d in (856, 264, 2056):
                # (more columns do not add a block of the first GEMM: both end in the same one)
                assert -(-f // 128) == -(-(f + 56) // 128)
                assert tile_us(experts, rows, d, f, gated, backward)[0] == \
                    tile_us(experts, rows, d, f + 56, gated, backward)[0]
