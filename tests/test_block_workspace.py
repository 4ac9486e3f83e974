"""CPU: the workspace of a block sweep has room for the records (64 bytes a thread block) of every
launch that the block's region may take: the default's, which may cut x into slabs of two planes
(162 blocks on 40^3 where a set tile has 9), and any tile set or tuned after the size was asked for."""
import ctypes
import math

import pytest

from paper_2604_25876_amd import skyr

HEAD, RECORD = 768, 64


@pytest.mark.parametrize("prec", [skyr.F64, skyr.F32_BULK])
@pytest.mark.parametrize("extent", [(1, 1, 1), (40, 40, 40), (128, 128, 128), (9, 700, 300), (300, 300, 300)])
def test_block_workspace_holds_every_launch(prec, extent):
    lat = skyr.Lattice((ctypes.c_int32 * 3)(*(e + 20 for e in extent)), 0, 0.2)
    blk = skyr.Block.of(lat, (8, 8, 8), extent)
    need = skyr.block_workspace_bytes(blk, prec)
    assert need >= HEAD + 4084 * RECORD  # the most blocks of a default launch
    # the tile of a block is that of a lattice whose interior is the block's region
    region = skyr.Lattice((ctypes.c_int32 * 3)(*(e + 4 for e in extent)), 0, 1.0)
    saved = skyr.get_tile(region, prec)
    try:
        for v, (_, oy, oz) in enumerate(skyr.tile_variants(prec)):
            for xc in (16, 64, 1000):
                skyr.set_tile(region, prec, v, xc)
                blocks = math.ceil(extent[0] / xc) * math.ceil(extent[1] / oy) * math.ceil(extent[2] / oz)
                assert skyr.block_workspace_bytes(blk, prec) == need >= HEAD + blocks * RECORD
    finally:
        skyr.set_tile(region, prec, *saved)
