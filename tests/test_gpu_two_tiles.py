"""bf16 at d = 64 with long lists: steps of two key tiles, a list of an odd length walks its last tile again and skips it."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from gpu_util import assert_close, oracle_rows, run_prefill

pytestmark = pytest.mark.gpu


def takes_two(tm, G):
    """The library's rule: twelve tiles per unit, or per workgroup where a launch has fewer units."""
    plan, n_wgs = tm.pair_plan(G), torch.cuda.get_device_properties(0).multi_processor_count
    return plan["unit_tiles"] >= 12 * max(plan["n_units"], n_wgs)


@pytest.mark.parametrize("flags", [0, bs.BS_MAP_REGROUP_ROWS, bs.BS_MAP_PACK_KEYS])
@pytest.mark.parametrize("kw", [{}, {"window": 1600}, {"img_bidir": True, "sink_offsets": (0, 5, 9)}])
@pytest.mark.parametrize("tail", [1, 60, 130])
def test_outputs(tail, kw, flags):
    rng = np.random.default_rng([tail, flags])
    classes = rng.integers(0, 4, 60)
    classes[:20] = 0   # whole groups of Dense heads: stacked rows
    p = W.custom_prompt([("T", 40), ("I", 1300), ("T", 9), ("I", 700), ("T", tail)], classes, 6, 64, dtype="bf16", sink_len=5,
                        value_recipe={"std": 1.0, "first_key_scale": 4.0}, name=f"two-{tail}", **kw)
    q, k, v = W.make_qkv(p, 7, "cuda:0")
    got, tm = run_prefill(p, q, k, v, flags=flags)
    assert takes_two(tm, 10)
    assert_close(got.float().cpu().numpy(), oracle_rows(p, q, k, v), "bf16", p.name)


@pytest.mark.parametrize("L,heads", [(1600, (64, 8)), (1601, (64, 8)), (1700, (64, 8)), (1792, (64, 8)), (1600, (320, 320))])
def test_last_tile_again(L, heads):
    """A score that is not a number in the last tile, of a key that only the last row sees: lists of 25 to 28 tiles, no unit cut.
    (Every wave of the last unit has a row that sees a key of that tile, so the scores are masked the first time.)"""
    p = W.custom_prompt([("T", L)], np.zeros(heads[0]), heads[1], 64, dtype="bf16", name=f"again-{L}")
    q, k, v = W.make_qkv(p, 8, "cuda:0")
    k[:, -1] = float("nan")
    got, tm = run_prefill(p, q, k, v)
    assert takes_two(tm, p.gqa_group)
    rows = np.arange(L - 140, L - 1, dtype=np.int32)
    part = W.custom_prompt([("T", L)], np.zeros(16), 16 * heads[1] // heads[0], 64, dtype="bf16", name="part")
    assert bool(torch.isfinite(got[:, :-1]).all())
    assert_close(got[:16, torch.from_numpy(rows).long()].float().cpu().numpy(), oracle_rows(part, q[:16], k[:part.n_kv_heads].nan_to_num(), v[:part.n_kv_heads], rows),
                 "bf16", p.name)


@pytest.mark.parametrize("L,heads", [(5938, 4), (4146, 8)])
def test_last_tile_again_in_parts(L, heads):
    """The same where most units are cut: the parts have odd lengths of their own, and the merge reads their row sums."""
    p = W.custom_prompt([("T", L)], np.zeros(heads), heads, 64, dtype="bf16", name=f"again-parts-{L}")
    q, k, v = W.make_qkv(p, 9, "cuda:0")
    k[:, -1] = float("nan")
    got, tm = run_prefill(p, q, k, v)
    plan = tm.share_plan(1, torch.cuda.get_device_properties(0).multi_processor_count)
    assert takes_two(tm, 1) and 2 * plan["n_cut_units"] > tm.pair_plan(1)["n_units"]
    assert bool(torch.isfinite(got[:, :-1]).all())
    rows = np.unique(np.concatenate([np.arange(0, L - 1, 61), np.arange(L - 140, L - 1)])).astype(np.int32)
    assert_close(got[:, torch.from_numpy(rows).long()].float().cpu().numpy(), oracle_rows(p, q, k.nan_to_num(), v, rows), "bf16", p.name)


@pytest.mark.parametrize("flags", [0, bs.BS_MAP_PACK_KEYS])
@pytest.mark.parametrize("image,text,dense,sink,n_kv", [(3000, 200, 12, 4, 4), (4000, 300, 24, 8, 8)])
def test_units_without_a_tile_beside_long_ones(image, text, dense, sink, n_kv, flags):
    """The image stands first and has no sinks, so its rows see nothing under the Sink heads; in equal shares and in queues."""
    p = W.custom_prompt([("I", image), ("T", text)], [0] * dense + [1] * sink, n_kv, 64, dtype="bf16", sink_len=0, span_sink=0, name=f"empty-{image}")
    q, k, v = W.make_qkv(p, 10, "cuda:0")
    got, tm = run_prefill(p, q, k, v, flags=flags)
    assert takes_two(tm, p.gqa_group) and tm.stats(1)["empty_rows"] == image
    rows = np.unique(np.concatenate([np.arange(0, p.seq_len, 47), [image - 1, image, p.seq_len - 1]])).astype(np.int32)
    out = got[:, torch.from_numpy(rows).long()].float().cpu().numpy()
    assert not out[dense:, rows < image].any()
    assert_close(out, oracle_rows(p, q, k, v, rows), "bf16", p.name)
