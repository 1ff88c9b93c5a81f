"""The list regions of the compression's one pass (host arithmetic, no GPU): every block has room in
proportion to the chunks it reads, regions follow each other and end inside the list."""
import ctypes

import pytest

import paper_2510_19470_amd as moe

CHUNK = 8192


@pytest.mark.parametrize("n", [
    1, 8192, 8193, 65537, 511 * CHUNK, 512 * CHUNK, 513 * CHUNK, 520 * CHUNK,   # 2080 x 2048
    576 * CHUNK, 1023 * CHUNK + 1, 1040 * CHUNK, 14336 * 4096, 2 ** 31 - 1])
@pytest.mark.parametrize("n_cu", [256, 304, 3])
def test_regions_are_proportional_to_chunks(n, n_cu):
    rule = moe.load_library().moe_internal_sr_region
    v = [ctypes.c_int64() for _ in range(4)]
    args = [ctypes.byref(x) for x in v]
    n_chunks = -(-n // CHUNK)
    blocks = rule(ctypes.c_int64(n), n_cu, 0, *args)
    share = v[3].value // n_chunks
    assert share * n_chunks > v[3].value - n_chunks      # less than an entry per chunk is lost
    end = chunks = 0
    for b in range(blocks):
        rule(ctypes.c_int64(n), n_cu, b, *args)
        own, first, entries, cap = (x.value for x in v)
        assert own == len(range(b, n_chunks, blocks))     # chunk c is read by block c modulo blocks
        assert entries == own * share and first == end
        end, chunks = first + entries, chunks + own
    assert chunks == n_chunks and end <= cap
