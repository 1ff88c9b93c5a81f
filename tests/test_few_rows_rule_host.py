"""When the expert FFN takes the kernel for few rows per expert (host arithmetic, no GPU).  The host
does not know how the tokens fall, so the rule has to hold when they all pick the same experts."""
import pytest

import paper_2510_19470_amd as moe

N_CU = 256


def few_rows(T, d, f, E, k, n_res, gated):
    return bool(moe.load_library().moe_internal_ffn_few_rows(T, d, f, E, k, n_res, int(gated), N_CU))


@pytest.mark.parametrize("T,d,f,E,k,n_res,gated", [
    # measured slower than the tiles when popularity falls off as rank^-1.2 or the tokens agree
    (200, 3072, 3072, 64, 6, 8, False), (48, 3072, 3072, 64, 6, 8, False),
    (200, 2048, 14336, 64, 2, 8, False), (32, 2048, 14336, 64, 2, 8, False),
    (200, 2048, 1408, 64, 6, 12, True), (96, 2048, 1408, 64, 6, 12, True),
    (120, 4096, 2048, 64, 2, 16, True), (30, 4096, 14336, 64, 4, 8, True),
    (16, 4096, 14336, 32, 2, 8, True), (200, 1024, 4096, 32, 2, 4, True),
    (96, 1024, 4096, 16, 2, 4, False),
    # ... than the 128-row tiles when the tokens agree or fall on the resident experts
    (64, 1024, 4096, 16, 2, 4, True), (64, 1024, 4096, 16, 2, 6, True), (48, 1024, 4096, 16, 2, 6, True),
    (24, 2048, 1408, 64, 6, 12, True), (32, 2048, 1408, 64, 6, 12, True), (8, 2048, 14336, 8, 2, 8, False)])
def test_left_to_the_tiles(T, d, f, E, k, n_res, gated):
    assert not few_rows(T, d, f, E, k, n_res, gated)


@pytest.mark.parametrize("T,d,f,E,k,n_res,gated", [
    # (within 2 %, one layer within 6 %, where the tokens fall on all the resident experts)
    (8, 1024, 4096, 16, 2, 6, True), (32, 1024, 4096, 16, 2, 6, True), (8, 3072, 3072, 64, 6, 8, False),
    (16, 2048, 1408, 64, 6, 12, True), (64, 768, 2048, 8, 2, 4, False), (2, 4096, 14336, 8, 2, 8, True),
    (32, 4096, 2048, 16, 2, 16, True), (64, 512, 1024, 32, 4, 8, True), (1, 8, 8, 4, 2, 4, True)])
def test_taken_where_it_is_no_slower_however_the_tokens_fall(T, d, f, E, k, n_res, gated):
    assert few_rows(T, d, f, E, k, n_res, gated)


def test_bounds_hold_for_every_routing():
    """At most one pass over an expert's weights (64 rows), at most 200 MB of token rows through L2, and no
    more than 48 KB per element of d where the 128-row tiles are the other choice."""
    tile128 = moe.load_library().moe_internal_ffn_tile128
    for d in (8, 512, 1024, 2048, 4096, 8192):
        for f in (8, 768, 4096, 14336):
            for E, k in ((4, 1), (8, 2), (64, 6), (256, 16)):
                for n_res in (1, E // 2, E):
                    for T in (1, 2, 8, 16, 47, 64, 65, 100, 200, 256):
                        if few_rows(T, d, f, E, k, n_res, True):
                            l2 = T * min(k, n_res) * d * f // 4
                            assert T <= 64 and l2 <= 200e6
                            assert l2 <= 48000 * max(d, 2048) or not tile128(T, d, f, E, k, n_res, 1, 0, N_CU)
