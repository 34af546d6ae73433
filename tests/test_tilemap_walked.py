"""The lists that the kernels walk where they differ from the published ones (text keys in compact tiles of their own, compact
tiles in a window): every allowed pair of the oracle's mask in exactly one tile, every state exact."""
import numpy as np
import pytest

import oracle
import paper_2507_09071_amd as bs
import workloads as W
from test_tilemap import packed_expectation
from test_tilemap_model import random_layout


def check_walked(tm, spans, L, sink_len, bm, bn, bidir, offsets, window=0):
    """Returns how many of the query tiles walk key tiles that the map does not publish."""
    imgid, issink = oracle.token_arrays(spans, L, sink_len, offsets)
    rows = tm.row_order(bm)
    n0, text, free = -(-L // bn), np.flatnonzero(imgid == 0), np.flatnonzero((imgid == 0) | (issink == 1))
    own_tiles = 0
    for c in range(4):
        full = oracle.mask(c, imgid, issink, bidir, window).astype(bool)
        for m in range(tm.n_q_tiles):
            states, keys, compact = tm.walked(c, m, bn)
            assert np.array_equal(keys[:n0].ravel()[:L], np.arange(L)) and (keys[:n0].ravel()[L:] < 0).all()
            # the tiles behind the prompt's: free keys, then (if they are there) text keys
            text0 = n0 + (-(-len(free) // bn) if len(states) > n0 else 0)
            assert len(states) in (text0, text0 + -(-len(text) // bn))
            assert np.array_equal(keys[n0:text0].ravel()[:len(free)], free[:bn * (text0 - n0)])
            assert np.array_equal(keys[text0:].ravel()[:len(text)], text[:bn * (len(states) - text0)])
            spaces = np.zeros(len(states), dtype=int)
            spaces[n0:text0], spaces[text0:] = 1, 2
            walks = {0} | ({2 if c == bs.INTRA and text0 < len(states) else 1} if compact else set())
            total = 0
            for n in range(len(states)):
                if spaces[n] not in walks:
                    assert states[n] == 0, (c, m, n)
                    continue
                cnt = int(packed_expectation(c, rows[m], keys[n], n < n0, full, imgid, compact, compact).sum())
                total += cnt
                assert states[n] == (0 if cnt == 0 else (2 if cnt == bm * bn else 1)), (c, m, n, states[n], cnt)
            assert total == int(full[rows[m][rows[m] >= 0]].sum()), (c, m)
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
            for window in (1, int(rng.integers(1, 20)), int(rng.integers(20, 90))):
                if window < L:
                    tw = bs.bs_build_tilemap(spans, L, classes, sink_len, bm, bn, sink_offsets=offsets, q_begin=q_begin, window=window,
                                             flags=bs.BS_MAP_PACK_KEYS | (bs.BS_MAP_BIDIR_IMAGES if bidir else 0))
                    check_walked(tw, spans, L, sink_len, bm, bn, bidir, offsets, window)
                    tw.pair_plan(2)
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


@pytest.mark.parametrize("bidir", [False, True])
@pytest.mark.parametrize("window", [100, 512, 1500])
def test_kernel_tile_size_window(window, bidir):
    runs = [("T", 9)]
    for i in range(14):
        runs += [("I", [64, 256, 333][i % 3]), ("T", 7 + i)]
    L, spans = W.layout_from_runs(runs, "prefix")
    offsets = [0, 3, 17, 64, 100, 200]
    tm = bs.bs_build_tilemap(spans, L, np.arange(8) % 4, 3, flags=bs.BS_MAP_PACK_KEYS | (bs.BS_MAP_BIDIR_IMAGES if bidir else 0),
                             window=window, sink_offsets=offsets)
    own = check_walked(tm, spans, L, 3, 128, 64, bidir, offsets, window)
    assert (own > 0) == (window > 100)   # (images of more than twice the window keep the published lists)


def test_units_of_two_heads_take_the_shorter_rule_block_by_block():
    """A Dense and a Sink head of one KV group in a window: image rows pair tiles of one head, text rows the two heads."""
    runs = [("T", 40)]
    for _ in range(40):
        runs += [("I", 256), ("T", 30)]
    L, spans = W.layout_from_runs(runs, "prefix")
    tm = bs.bs_build_tilemap(spans, L, [bs.DENSE, bs.SINK], 3, flags=bs.BS_MAP_PACK_KEYS | bs.BS_MAP_BIDIR_IMAGES, window=1024,
                             sink_offsets=list(range(0, 256, 9)))
    M = tm.n_q_tiles
    visited = [[tm.walked(c, m)[0] > 0 for m in range(M)] for c in (bs.DENSE, bs.SINK)]
    blocks = [range(m, min(m + 2, M)) for m in range(0, M, 2)]
    rows = [sum(int(np.any([v[m] for m in b], axis=0).sum()) for v in visited) for b in blocks]
    cross = [sum(int((visited[0][m] | visited[1][m]).sum()) for m in b) for b in blocks]
    steps = tm.pair_plan(2)["unit_tiles"]
    assert sum(np.minimum(rows, cross)) <= steps < 0.95 * min(sum(rows), sum(cross))


@pytest.mark.parametrize("seed", range(12))
def test_tiles_that_no_list_walks_are_not_there(seed):
    """The workspace of a call has room for every tile that the kernels know."""
    rng = np.random.default_rng([5, seed])
    spans, pos, L = [], 9, 9000
    while pos + 1500 < L:
        n = int(rng.integers(64, [200, 600, 1500][seed % 3]))
        spans.append((pos, pos + n, max(1, n // 10)))
        pos += n + int(rng.integers(4, 64))
    for window in (0, 256, 1024):
        for bidir in (False, True):
            tm = bs.bs_build_tilemap(spans, L, np.arange(4), 5, window=window, q_begin=int(rng.choice([0, L - 300])),
                                     flags=bs.BS_MAP_PACK_KEYS | (bs.BS_MAP_BIDIR_IMAGES if bidir else 0))
            states = {c: np.array([tm.walked(c, m)[0] for m in range(tm.n_q_tiles)]) for c in (bs.SINK, bs.INTRA, bs.INTRA_SINK)}
            known, n_text = states[bs.SINK].shape[1], -(-(L - sum(e - s for s, e, _ in spans)) // 64)
            more = {c: bool((states[c][:, tm.n_k_tiles:] > 0).any()) for c in states}
            assert (known > tm.n_k_tiles) == any(more.values())
            if window and known > tm.n_k_tiles and not more[bs.INTRA]:   # free keys alone
                n_free = L - sum(e - s - k for s, e, k in spans)
                assert known == tm.n_k_tiles + -(-n_free // 64)
            elif not window and known > tm.n_k_tiles:
                assert known == tm.n_k_tiles + n_text
