"""The tiles that bench.py counts are those that the kernels walk."""
import numpy as np
import pytest

import bench
import paper_2507_09071_amd as bs


@pytest.mark.parametrize("window", [0, 1024])
def test_tiles_of_a_launch(window):
    spans = [(p, p + 256, 26) for p in range(20, 9000, 276)]
    classes = np.array([0, 1, 2, 3, 3, 2, 1, 1], dtype=np.uint8)
    tm = bs.bs_build_tilemap(spans, 9300, classes, 5, flags=bs.BS_MAP_PACK_KEYS, window=window)
    tot, _ = bench.class_totals(tm, classes)
    states = [np.array([tm.walked(c, m)[0] for m in range(tm.n_q_tiles)]) for c in range(4)]
    assert tot["visited"] == sum(int((states[c] > 0).sum()) for c in classes)
    assert tot["full"] == sum(int((states[c] == 2).sum()) for c in classes) and tot["partial"] == tot["visited"] - tot["full"]
    assert tot["visited"] < sum(tm.stats(int(c))["visited"] for c in classes)     # fewer than published: text tiles, windows
    assert tot["allowed_pairs"] == sum(tm.stats(int(c))["allowed_pairs"] for c in classes)
    plan = tm.pair_plan(2)   # a step of a unit serves one item or two
    assert 2 * plan["unit_tiles"] - plan["skip_steps"] == tot["visited"]
