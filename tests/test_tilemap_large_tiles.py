"""Query tiles longer than the prompt, up to the largest number that the argument holds: one tile per group of rows, as with a tile
of just the prompt's length."""
import numpy as np
import pytest

import paper_2507_09071_amd as bs

SPANS, L, CLASSES = [(10, 200, 5), (300, 800, 0)], 1000, [0, 1, 2, 3]


@pytest.mark.parametrize("flags", [0, bs.BS_MAP_REGROUP_ROWS, bs.BS_MAP_PACK_KEYS])
@pytest.mark.parametrize("q_begin", [0, 350, 999])
@pytest.mark.parametrize("block_m", [2 ** 31 - 1, 2 ** 31 - 500, 2 ** 30 + 1])
def test_tile_longer_than_the_prompt(block_m, q_begin, flags):
    # (the row order has one entry per row of a tile: not asked for here)
    big, small = (bs.bs_build_tilemap(SPANS, L, CLASSES, 4, bm, 64, flags=flags, q_begin=q_begin) for bm in (block_m, 1024))
    assert big.n_q_tiles == small.n_q_tiles >= 1 and big.n_k_tiles == small.n_k_tiles
    for c in range(4):
        assert big.stats(c) == small.stats(c)
        assert np.array_equal(big.tile_states(c), small.tile_states(c))
