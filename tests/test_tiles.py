"""Tile counts on the host at the largest joins (two sides of 2^31 - 1 rows are
2^32 - 2 records): no count wraps, so every record has a tile (no GPU needed)."""
import ctypes

import pytest

from paper_1702_03484_amd import binding

MOST = 2**32 - 2


def native(symbol, res, *args):
    fn = getattr(ctypes.CDLL(binding.LIB_PATH), symbol)
    fn.restype, fn.argtypes = res, args
    return fn


@pytest.mark.parametrize("gen", [False, True])
@pytest.mark.parametrize("kpt", [8, 16])
@pytest.mark.parametrize("rb", [4, 8, 9, 11])
def test_radix_tiles(rb, kpt, gen):
    tiles = native("_ZN2mq11radix_tilesEjiib", ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int, ctypes.c_int,
                   ctypes.c_bool)
    tile = 2**31 // tiles(2**31, kpt, rb, gen)
    for n in (2**31 + 1, 2**32 - 40_000, 2**32 - tile - 1, 2**32 - tile, 2**32 - tile + 1, MOST - 1, MOST):
        assert tiles(n, kpt, rb, gen) == -(-n // tile), n
    assert tiles(0, kpt, rb, gen) == 0 and tiles(1, kpt, rb, gen) == 1


@pytest.mark.parametrize("brk", [False, True])
def test_segment_scratch(brk):
    size = native("_ZN2mq17seg_scratch_bytesEjb", ctypes.c_size_t, ctypes.c_uint32, ctypes.c_bool)
    # 2^20 tiles of 4,096 records either way: what the largest join needs is what 2^32 - 4,096 records do
    assert size(MOST, brk) >= size(2**32 - 4096, brk) > size(2**31, brk) > size(4096, brk) > 0
