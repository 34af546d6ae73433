"""GPU parity where the launch hands out equal shares of cut units instead of queued ones (few units for the chip): chunks
behind a long cache, short prompts, an odd head left alone, items whose parts hold no visible key for some rows."""
import numpy as np
import pytest

import paper_2507_09071_amd as bs
import workloads as W
from test_gpu_model import suffix_parity
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
D, S, I, IS = 0, 1, 2, 3
RUNS = [("T", 40), ("I", 900), ("T", 20), ("I", 1500), ("T", 9), ("I", 333), ("T", 12), ("I", 700), ("T", 77)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows", [33, 128, 129, 517, 1000])
def test_chunk_behind_a_cache(rows, d):
    p = W.custom_prompt(RUNS, [D, S, I, IS, IS, I, S], 1, d, dtype="bf16", sink_len=40, name=f"shares-chunk{rows}-d{d}",
                        value_recipe={"std": 1.0, "first_key_scale": 4.0})
    suffix_parity(p, p.seq_len - rows, 51, bs.BS_MAP_PACK_KEYS, row_step=3)


@pytest.mark.parametrize("classes,n_kv", [([D], 1), ([IS, I, S], 1), ([D, D, I, S, IS, IS, D, D], 4)])
@pytest.mark.parametrize("flags", [0, bs.BS_MAP_REGROUP_ROWS, bs.BS_MAP_PACK_KEYS])
def test_short_prompt(classes, n_kv, flags):
    runs = [("I", 300), ("T", 3), ("I", 410), ("T", 50), ("I", 128), ("T", 5)]   # image first: rows without a visible key
    p = W.custom_prompt(runs, classes, n_kv, 128, dtype="bf16", sink_len=0, span_sink=0, name=f"shares-short-f{flags}")
    full_parity(p, seed=52, flags=flags)


def test_window_and_bidirectional_images():
    p = W.custom_prompt(RUNS, [D, S, I, IS], 2, 128, dtype="bf16", sink_len=3, span_sink=0, name="shares-window",
                        img_bidir=True, sink_offsets=(0, 5, 64, 130, 299), window=500)
    suffix_parity(p, p.seq_len - 700, 53, bs.BS_MAP_REGROUP_ROWS, row_step=5)
