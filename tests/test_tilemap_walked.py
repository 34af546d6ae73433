"""The lists that the kernels walk where they differ from the published ones (text keys in compact tiles of their own): every
allowed pair of the oracle's mask in exactly one tile, every state exact."""
import numpy as np
import pytest

import oracle
import paper_2507_09071_amd as bs
import workloads as W
from test_tilemap import packed_expectation
from test_tilemap_model import random_layout


def check_walked(tm, spans, L, sink_len, bm, bn, bidir, offsets, q_tiles=None, window=0):
    """Returns how many of the query tiles walk key tiles that the map does not publish."""
    imgid, issink = oracle.token_arrays(spans, L, sink_len, offsets)
    rows = tm.row_order(bm)
    own_tiles = 0
    for c in range(4):
        for m in range(tm.n_q_tiles) if q_tiles is None else q_tiles:
            states, keys, compact = tm.walked(c, int(m), bn)
            n0 = -(-L // bn)
            assert np.array_equal(keys[:n0].ravel()[:L], np.arange(L)) and (keys[:n0].ravel()[L:] < 0).all()
            valid = rows[m][rows[m] >= 0]
            allowed = oracle.mask_rows(c, imgid, issink, valid, bidir, window)
            mask = np.zeros((L, L), dtype=bool) if L <= 4000 else None
            if mask is not None:
                mask[valid] = allowed
            total = 0
            for n in range(len(states)):
                if states[n] == 0 and n >= n0 and not compact:
                    continue
                if states[n] == 0 and n >= tm.n_k_tiles and c != bs.INTRA:
                    continue   # (tiles of the text keys alone, which only Intra-Image walks)
                if c == bs.INTRA and len(states) > tm.n_k_tiles and n0 <= n < tm.n_k_tiles:
                    assert states[n] == 0   # (its text keys are in the tiles behind)
                    continue
                cnt = int(packed_expectation(c, rows[m], keys[n], n < n0, mask, imgid, compact, compact).sum())
                total += cnt
                assert states[n] == (0 if cnt == 0 else (2 if cnt == bm * bn else 1)), (c, m, n, states[n], cnt)
            assert total == int(allowed.sum()), (c, m)
            own_tiles += int((states[tm.n_k_tiles:] > 0).any())
    return own_tiles


@pytest.mark.parametrize("seed", range(60))
def test_random_prompts(seed):
    L, spans, offsets, sink_len, bm, bn = random_layout(900 + seed, equal_images=seed % 2 == 0)
    if not L:
        return
    rng = np.random.default_rng(seed)
    classes = rng.integers(0, 4, 6).astype(np.uint8)
    for bidir in (False, True):
        for q_begin in (0, int(rng.integers(0, L))):
            tm = bs.bs_build_tilemap(spans, L, classes, sink_len, bm, bn, sink_offsets=offsets, q_begin=q_begin,
                                     flags=bs.BS_MAP_PACK_KEYS | (bs.BS_MAP_BIDIR_IMAGES if bidir else 0))
            check_walked(tm, spans, L, sink_len, bm, bn, bidir, offsets)
            for group in (1, 2, 3):
                tm.pair_plan(group)
            tm.share_plan(2, 7)
            tm.share_plan(0, 7)


@pytest.mark.parametrize("text", [1, 17, 64, 130])
def test_kernel_tile_size(text):
    runs = [("T", text)]
    for i in range(9):
        runs += [("I", [64, 200, 333][i % 3]), ("T", text)]
    L, spans = W.layout_from_runs(runs, "paper10")
    tm = bs.bs_build_tilemap(spans, L, np.arange(8) % 4, 3, flags=bs.BS_MAP_PACK_KEYS)
    own = check_walked(tm, spans, L, 3, 128, 64, False, None)
    n_text = -(-text * 10 // 64)
    assert (own > 0) == (2 * n_text + 1 <= -(-L // 64)) and len(tm.walked(0, 0)[0]) == tm.n_k_tiles + (n_text if own else 0)
