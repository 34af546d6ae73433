"""Equal shares on the host: bs_tilemap_share_plan answers BS_OK only if every unit has a part, the parts of a unit walk each of
its key tiles once and every part's slot is named in the list of cut items."""
import numpy as np
import pytest

import paper_2507_09071_amd as bs
import workloads as W

D, S, I, IS = 0, 1, 2, 3
CUS = 256


@pytest.mark.parametrize("seq_len", [38656, 38784, 39168])
def test_units_without_a_key_tile_bidirectional(seq_len):
    """One image without sinks: the rows of the Sink heads see nothing, but somebody has to write their zeros."""
    tm = bs.bs_build_tilemap([(0, seq_len - 7, 0)], seq_len, [D, D, S, S], 0, 128, 64,
                             flags=bs.BS_MAP_BIDIR_IMAGES | bs.BS_MAP_REGROUP_ROWS)
    assert tm.share_plan(4, CUS)["n_queued"] > 0


def test_units_without_a_key_tile_window():
    tm = bs.bs_build_tilemap([(0, 141000, 0)], 141000, [D] * 28 + [S] * 4, 0, 128, 64, window=32768, q_begin=141000 - 2816)
    assert tm.stats(S)["empty_rows"] == 2816
    assert tm.share_plan(8, CUS)["n_queued"] > 0


@pytest.mark.parametrize("rows,n_kv,G,L,queued", [(1, 4, 7, 39500, False), (128, 4, 7, 36864, False), (517, 4, 7, 36864, False),
                                                  (2048, 8, 5, 140997, True), (1500, 4, 7, 150000, True)])
def test_chunk_behind_a_cache(rows, n_kv, G, L, queued):
    rng = np.random.default_rng(L)
    pos, spans = 64, []
    while pos < L - 4000:
        n = int(rng.integers(64, 3600))
        spans.append((pos, pos + n, (n + 9) // 10))
        pos += n + int(rng.integers(8, 65))
    tm = bs.bs_build_tilemap(spans, L, rng.permutation(np.arange(n_kv * G) % 4), 64, 128, 64, flags=bs.BS_MAP_PACK_KEYS,
                             q_begin=L - rows)
    plan = tm.share_plan(G, CUS)
    assert plan["n_parts"] > 0 and plan["n_cut_units"] > 0
    assert (plan["n_queued"] > 0) == queued   # long shares keep back a part of the steps for the queues


@pytest.mark.parametrize("seed", range(60))
def test_random_prompts(seed):
    rng = np.random.default_rng([11, seed])
    runs = [(("T", "I")[i % 2], int(np.exp(rng.uniform(0, np.log([300, 20000][i % 2]))))) for i in range(int(rng.integers(1, 14)))]
    if rng.random() < 0.5:
        runs = runs[1:] or runs   # image first
    L, spans = W.layout_from_runs(runs, span_sink=int(rng.choice([0, 0, 7])))
    n_kv, G = int(rng.choice([1, 2, 4, 8])), int(rng.choice([1, 2, 5, 7]))
    flags = int(rng.choice([0, bs.BS_MAP_REGROUP_ROWS, bs.BS_MAP_PACK_KEYS])) | int(rng.choice([0, bs.BS_MAP_BIDIR_IMAGES]))
    tm = bs.bs_build_tilemap(spans, L, rng.integers(0, 4, n_kv * G), int(rng.choice([0, min(L, 5)])), 128, 64, flags=flags,
                             window=int(rng.choice([0, 0, 512, 5000])), q_begin=int(rng.choice([0, L // 2, L - 1])))
    for wgs in (CUS, 2 * CUS, 7):
        tm.share_plan(G, wgs)
        tm.share_plan(0, wgs)   # the fp32 kernel's units


def test_refuses_what_it_cannot_plan():
    tm = bs.bs_build_tilemap([(10, 200, 5)], 300, [D, S, I, IS], 4, 128, 64)
    for group, wgs in ((3, CUS), (-1, CUS), (2, 0)):
        with pytest.raises(bs.BlindsightError):
            tm.share_plan(group, wgs)


def test_units_of_another_group_size_in_between():
    """The shares are there already, but the units that they are cut from have been planned for other groups since."""
    spans = [(p, p + 1000, 100) for p in range(20, 36000, 1018)]
    tm = bs.bs_build_tilemap(spans, 36660, np.arange(16) % 4, 5, 128, 64, flags=bs.BS_MAP_PACK_KEYS, q_begin=36660 - 517)
    plan = tm.share_plan(4, CUS)
    assert plan["n_parts"] > 0
    tm.pair_plan(8)
    assert tm.share_plan(4, CUS) == plan
