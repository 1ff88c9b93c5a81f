"""When the expert FFN takes 128-row tiles, and the workspace of their cut contractions (host arithmetic,
no GPU).  The host does not know how the tokens fall: the rule goes by an even routing and by one where all
tokens agree."""
import ctypes

import pytest

import paper_2510_19470_amd as moe

N_CU = 256


def tile128(T, d, f, E, k, n_res, gated, backward):
    return bool(moe.load_library().moe_internal_ffn_tile128(T, d, f, E, k, n_res, int(gated), int(backward), N_CU))


def tile_us(experts, rows, d, f, gated, backward):
    us = (ctypes.c_double * 2)()
    moe.load_library().moe_internal_ffn_tile_us(experts, rows, d, f, int(gated), int(backward), N_CU, us)
    return us[0], us[1]


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


@pytest.mark.parametrize("T,d,f,E,k,n_res,gated,backward", [
    # measured faster with the smaller tiles evenly, but up to 1.5 times slower where the tokens agree: d > f,
    # the second GEMM has the more tiles
    (953, 4096, 1024, 64, 8, 12, True, False), (5765, 2816, 896, 16, 3, 3, True, False),
    (2999, 3328, 1280, 64, 8, 8, True, True), (2615, 3840, 768, 64, 3, 22, True, False),
    # ... and where both have about as many
    (1000, 3072, 3072, 64, 6, 10, False, False), (1000, 3072, 3072, 64, 6, 10, False, True),
    (1441, 4096, 4352, 16, 1, 4, True, False), (2282, 1536, 1024, 32, 5, 16, True, True),
    # slower with any routing
    (2166, 1792, 1408, 32, 4, 16, False, True), (343, 3840, 14080, 8, 2, 3, True, True),
    (1422, 1816, 2672, 8, 3, 3, True, False), (64, 4096, 14336, 8, 2, 8, True, True)])
def test_rule_looks_at_both_gemms_and_at_tokens_that_agree(T, d, f, E, k, n_res, gated, backward):
    assert not tile128(T, d, f, E, k, n_res, gated, backward)


@pytest.mark.parametrize("T,d,f,E,k,n_res,gated,backward,want", [
    # near the line; evenly routed, larger tiles (backward: dH by turn) -> smaller ones, us
    (275, 4096, 4480, 8, 3, 8, True, False, True),       # 247 -> 204
    (7513, 1536, 1536, 32, 1, 9, False, False, True),    # 80 -> 50
    (1422, 1816, 2672, 8, 3, 3, True, False, False),     # 95 -> 100
    (5102, 1976, 320, 32, 5, 16, True, False, False),    # 97 -> 106
    (417, 2304, 3072, 64, 1, 19, True, True, True),      # 177 -> 153
    (337, 3328, 2816, 32, 2, 14, True, True, True),      # 170 -> 154
    (338, 3840, 3712, 64, 1, 16, True, True, True),      # 234 -> 209
    (7216, 1280, 768, 8, 3, 4, False, True, False),      # 81 -> 91
    (4778, 2048, 896, 16, 1, 11, True, True, False),     # 90 -> 94
    (901, 2816, 896, 32, 6, 14, True, True, False),      # 104 -> 109
])
def test_rule_near_the_line(T, d, f, E, k, n_res, gated, backward, want):
    assert tile128(T, d, f, E, k, n_res, gated, backward) == want


def test_estimate_cuts_gate_up_as_the_kernel_does():
    """Few tiles and a long contraction: the smaller tiles' gate/up is cut (8 parts of 64 steps), dH is not."""
    parts = moe.load_library().moe_internal_tile128_parts(2, 2 * N_CU, 64)
    assert parts == 8
    forward = tile_us(1, 64, 4096, 128, True, False)[1]
    backward = tile_us(1, 64, 4096, 256, False, True)[1]     # dH: two tiles of 64 steps as well
    assert forward < backward - 20


@pytest.mark.parametrize("backward", [False, True])
def test_tokens_that_agree_cost_no_more_than_twice_the_gain(backward):
    taken = 0
    for d in (8, 512, 2048, 4096):
        for f in (8, 768, 4096, 14336):
            for E, k in ((4, 1), (8, 2), (64, 6), (256, 16)):
                for n_res in (1, E // 2, E):
                    for T in (129, 200, 1000, 4096, 16384, 200000):
                        for gated in (True, False):
                            if tile128(T, d, f, E, k, n_res, gated, backward):
                                large, small = tile_us(n_res, -(-T * k // E), d, f, gated, backward)
                                large_hot, small_hot = tile_us(min(k, n_res), T, d, f, gated, backward)
                                assert 0 < large - small and small_hot - large_hot <= 2 * (large - small) + 5
                                taken += 1
    assert taken > 100


@pytest.mark.parametrize("slots", [16, 512, 608])
def test_parts_fit_the_resident_blocks(slots):
    parts = moe.load_library().moe_internal_tile128_parts
    for kt in (1, 7, 8, 9, 16, 63, 64, 448):
        most = parts(1, 8, kt)                  # what the workspace is sized with
        assert (most == 1) == (kt < 8)
        for tiles in list(range(0, 70)) + [127, 128, 255, 256, 257, 512, 5000]:
            n = parts(tiles, slots, kt)
            assert 1 <= n <= most and (n == 1 or (tiles * n <= slots and kt // n >= 4))


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


@pytest.mark.parametrize("n_cu", [8, 256, 304])
def test_partial_sums_fit_the_workspace(n_cu):
    """Every launch that a context can make, forward and both dX contractions, against what moe_create
    allocates for it."""
    lib = moe.load_library()
    lib.moe_internal_tile128_split_floats.restype = ctypes.c_int64
    slots, cut = max(8, 2 * n_cu // 8 * 8), 0
    for S in (0, 1, 100, 128, 129, 1000, 20000):
        for E in (1, 3, 8, 256):
            for d in (8, 128, 136, 1160, 4096):
                for f in (8, 128, 192, 200, 256, 448, 520, 2888):
                    have = lib.moe_internal_tile128_split_floats(S, E, d, f, n_cu)
                    steps, cols = -(-f // 64), -(-d // 128)
                    most_blocks = S // 128 + E      # what the kernel counts up to
                    for blocks in {1, 2, 3, 7, 8, E, most_blocks // 2, most_blocks - 1, most_blocks}:
                        if not 1 <= blocks <= most_blocks:
                            continue
                        for kt in (steps, 2 * steps):
                            parts = lib.moe_internal_tile128_parts(blocks * cols, slots, kt)
                            if parts > 1:
                                assert blocks * cols * parts * 128 * 128 <= have
                                cut += 1
                    assert have <= slots * 128 * 128
    assert cut > 1000


@pytest.mark.parametrize("n_cu", [8, 256, 304])
def test_every_cut_gemm_fits_the_workspace_and_the_counters(n_cu):
    """Gate/up of the gated expert (64 columns a tile) and of the two-matrix one, down and both dX contractions, with
    tiles that share their weights or not: the partial tiles fit what moe_create allocates, and there are counters
    for slots / 2 tiles."""
    lib = moe.load_library()
    lib.moe_internal_tile128_split_floats.restype = ctypes.c_int64
    slots, cut = max(8, 2 * n_cu // 8 * 8), set()
    for S in (0, 1, 127, 128, 1000, 20000):
        for E in (1, 3, 40, 256):
            for d in (8, 136, 512, 1160, 4096, 14336):
                for f in (8, 64, 200, 512, 2888, 14336):
                    have = lib.moe_internal_tile128_split_floats(S, E, d, f, n_cu)
                    kd, kf = -(-d // 64), -(-f // 64)
                    for name, kt, cols in (("gate/up", kd, kf), ("up", kd, -(-f // 128)), ("down", kf, -(-d // 128)),
                                           ("dX", 2 * kf, -(-d // 128))):
                        most = S // 128 + E                      # row blocks that the kernel counts up to
                        for blocks in {1, 2, 3, 5, E, most // 2, most}:
                            if not 1 <= blocks <= most:
                                continue
                            for parts_of in (lib.moe_internal_tile128_parts, lib.moe_internal_tile128_parts_shared):
                                parts = parts_of(blocks * cols, slots, kt)
                                if parts > 1:
                                    assert blocks * cols * parts * 128 * 128 <= have
                                    assert blocks * cols <= slots // 2 and parts <= 8
                                    cut.add((name, parts))
    assert {name for name, _ in cut} == {"gate/up", "up", "down", "dX"} and {n for _, n in cut} >= {2, 3, 4, 5, 8}
