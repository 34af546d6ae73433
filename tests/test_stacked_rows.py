"""Query tiles that hold the rows of all heads of a KV group: text rows, and all rows where every head is Dense."""
import numpy as np
import pytest

import paper_2507_09071_amd as bs
import workloads as W

D, S, I, IS = 0, 1, 2, 3


def spans_of(rng, L, lo, hi, text):
    spans, pos = [], int(rng.integers(0, 40))
    while pos + hi + text < L:
        n = int(rng.integers(lo, hi))
        spans.append((pos, pos + n, n // 10))
        pos += n + int(rng.integers(0, text))
    return spans


@pytest.mark.parametrize("seed", range(40))
def test_units_of_random_prompts(seed):
    """pair_plan answers only if every row of every head is in one unit and a stacked tile's states are those of its rows."""
    rng = np.random.default_rng([21, seed])
    L = int(rng.integers(300, 9000))
    G, n_kv = int(rng.choice([2, 3, 5, 7, 16])), int(rng.choice([1, 2]))
    spans = spans_of(rng, L, 30, int(rng.choice([200, 2000])), int(rng.choice([20, 200])))
    flags = int(rng.choice([0, bs.BS_MAP_REGROUP_ROWS, bs.BS_MAP_PACK_KEYS])) | int(rng.choice([0, bs.BS_MAP_BIDIR_IMAGES]))
    tm = bs.bs_build_tilemap(spans, L, rng.integers(0, 4, G * n_kv), 5, 128, 64, flags=flags, window=int(rng.choice([0, 0, 70, 700])),
                             q_begin=int(rng.choice([0, L // 2, max(0, L - 130), L - 1])))
    for classes in (None, np.zeros(G * n_kv), np.repeat([0, 3], [G, G * (n_kv - 1)])):
        if classes is not None:
            tm.rebind(classes.astype(np.uint8))
        tm.pair_plan(G)
        tm.share_plan(G, 256)


def test_few_text_rows_are_a_fraction_of_the_units():
    spans = [(p, p + 1000, 100) for p in range(20, 36000, 1018)]
    L, q_begin = spans[-1][1] + 18, spans[-3][1] + 9
    tm = bs.bs_build_tilemap(spans, L, np.full(32, IS), 5, 128, 64, flags=bs.BS_MAP_PACK_KEYS, q_begin=q_begin)
    steps = [int((tm.walked(IS, m)[0] > 0).sum()) for m in range(tm.n_q_tiles)]
    text_rows = L - q_begin - 2000
    assert text_rows == 45 and tm.n_q_tiles == 17             # sixteen tiles of image rows, one that is a third full
    units = -(-(-(-8 * text_rows // 128)) // 2)               # of a group of eight heads; four otherwise
    assert units == 2
    assert tm.pair_plan(8)["unit_tiles"] <= 16 * sum(steps[:-1]) + 4 * units * steps[-1] < 16 * sum(steps)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,text,rows", [(3, 43, 0), (3, 128, 0), (7, 18, 300), (7, 19, 37), (5, 26, 129), (8, 64, 700), (33, 20, 64)])
def test_outputs(G, text, rows, d):
    from gpu_util import assert_close
    from test_gpu_model import suffix_parity
    from test_gpu_parity import full_parity
    classes = np.random.default_rng([G, text]).integers(0, 4, 2 * G)
    classes[G:] = 0   # the second group: every row stacked
    runs = [("T", text), ("I", 300), ("T", 2), ("I", 260), ("I", 150), ("T", text - 2), ("I", 222), ("T", 1)]
    for kw in ({}, {"window": 200}, {"img_bidir": True, "sink_offsets": (0, 5, 9)}):
        p = W.custom_prompt(runs, classes, 2, d, dtype="bf16", sink_len=5, name=f"stacked-{G}-{text}-{rows}", **kw)
        for flags in (bs.BS_MAP_PACK_KEYS, bs.BS_MAP_REGROUP_ROWS, 0):
            if rows:
                suffix_parity(p, p.seq_len - rows, 31, flags | (bs.BS_MAP_BIDIR_IMAGES if kw.get("img_bidir") else 0))
            else:
                full_parity(p, seed=31, flags=flags)
