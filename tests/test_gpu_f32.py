"""GPU parity of the fp32 kernel: one item per workgroup and equal shares of cut items, both head dimensions, ragged last
tiles, compact tiles (gathered keys), one tile and many, chunks, windows."""
import numpy as np
import pytest

import paper_2507_09071_amd as bs
import workloads as W
from test_gpu_model import suffix_parity
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
D, S, I, IS = 0, 1, 2, 3


def prompt(L, classes, n_kv, d, **kw):
    runs, left = [("T", min(L, 9))], L - min(L, 9)
    while left > 60:
        n = min(400, left - 30)
        runs += [("I", n), ("T", min(20, left - n))]
        left -= n + min(20, left - n)
    runs.append(("T", left))
    return W.custom_prompt(runs, classes, n_kv, d, dtype="f32", sink_len=min(3, L), name=f"f32-L{L}-d{d}",
                           value_recipe={"std": 1.0, "first_key_scale": 2.0}, **kw)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [1, 63, 64, 65, 129, 1000])
def test_lengths(L, d):
    full_parity(prompt(L, [D, S, I, IS, S, D], 2, d), seed=61, flags=bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("d,heads,L", [(64, 240, 700), (128, 160, 600)])
def test_more_items_than_shares_are_made_for(d, heads, L):
    """Some thousand items: one workgroup per item, nothing is cut."""
    full_parity(prompt(L, np.arange(heads) % 4, 8, d), seed=62, flags=bs.BS_MAP_REGROUP_ROWS)


@pytest.mark.parametrize("rows", [1, 130, 500])
@pytest.mark.parametrize("flags", [0, bs.BS_MAP_PACK_KEYS])
def test_chunks(rows, flags):
    p = prompt(2500, [D, S, I, IS], 2, 128)
    suffix_parity(p, p.seq_len - rows, 63, flags, row_step=3)


def test_window_and_bidirectional_images():
    p = prompt(1500, [D, S, I, IS], 2, 64, img_bidir=True, sink_offsets=(0, 5, 64, 130, 299), window=200)
    full_parity(p, seed=64, flags=bs.BS_MAP_REGROUP_ROWS)
