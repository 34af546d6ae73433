"""The prompt's complete K tiles are read where the caller has them, a ragged last one and the compact tiles from packed copies: prompt
lengths around multiples of the 64-key tile, with and without compact tiles, tiles fetched a few times and often, in windows and for chunks."""
import numpy as np
import pytest

import paper_2507_09071_amd as bs
import workloads as W
from test_gpu_model import suffix_parity
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu


def prompt(L, n_kv, G, d, **kw):
    runs, left = [("T", 7)], L - 7
    while left > 60:
        n = min(333, left - 20)
        runs += [("I", n), ("T", min(13, left - n))]
        left -= n + min(13, left - n)
    if left > 0:
        runs.append(("T", left))
    return W.custom_prompt(runs, np.arange(n_kv * G) % 4, n_kv, d, dtype="bf16", sink_len=5, name=f"in-place-L{L}-d{d}",
                           value_recipe={"std": 1.0, "first_key_scale": 4.0}, **kw)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("flags", [0, bs.BS_MAP_PACK_KEYS])
@pytest.mark.parametrize("L", [40, 63, 64, 65, 127, 128, 129, 640, 1000])
def test_few_fetches(L, flags, d):
    full_parity(prompt(L, 2, 2, d), seed=71, flags=flags)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [6, 8, 10, 12])   # some 32 to 60 fetches per tile, 40 complete ones and one of 40 keys
def test_many_fetches(G, d):
    full_parity(prompt(2600, 1, G, d), seed=72, flags=bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("rows", [100, 640])
def test_chunk_in_a_window(rows):
    p = prompt(4160, 2, 2, 128, window=500)
    suffix_parity(p, p.seq_len - rows, 73, bs.BS_MAP_REGROUP_ROWS, row_step=7)
