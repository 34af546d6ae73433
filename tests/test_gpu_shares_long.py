"""GPU parity of equal shares whose workgroups are handed more than 600 steps: the parts that are left to the queues, and units
without a key tile (an image without sinks under a Sink head: rows of zeros)."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from gpu_util import assert_close, oracle_rows
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu
D, S, I, IS = 0, 1, 2, 3


def parity(p, q_begin, seed, flags, n_rows):
    """Every element of the result is written; `n_rows` rows agree with the oracle."""
    q, k, v = W.make_qkv(p, seed, DEV)
    tm = bs.bs_build_tilemap(p.spans, p.seq_len, p.head_class, p.sink_len, 128, 64, window=p.window, q_begin=q_begin,
                             flags=flags | (bs.BS_MAP_BIDIR_IMAGES if p.img_bidir else 0))
    assert tm.share_plan(p.gqa_group, torch.cuda.get_device_properties(0).multi_processor_count)["n_queued"] > 0
    qs = q[:, q_begin:].contiguous()
    out = torch.full_like(qs, float("nan"))
    print(p.name, "L", p.seq_len, "q_begin", q_begin, flush=True)
    bs.bs_attn_prefill(qs, k, v, out, tm, bs.BS_BF16, p.n_q_heads, p.gqa_group, p.head_dim, p.scale,
                       torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out).all())
    rows = np.unique(np.linspace(q_begin, p.seq_len - 1, n_rows).astype(np.int32))
    want = oracle_rows(p, q, k, v, rows)
    got = out[:, torch.from_numpy(rows - q_begin).long().to(out.device)].float().cpu().numpy()
    for h in range(p.n_q_heads):
        assert_close(got[h], want[h], "bf16", f"{p.name} head {h}")
    return out


@pytest.mark.parametrize("d", [64, 128])
def test_chunk_with_parts_for_the_queues(d):
    runs = [("T", 40)] + [("I", 3500), ("T", 30)] * 33 + [("T", 77)]
    p = W.custom_prompt(runs, [D, D, S, D, I, D, IS, D], 1, d, dtype="bf16", sink_len=40, name=f"shares-queued-d{d}",
                        value_recipe={"std": 1.0, "first_key_scale": 4.0})
    parity(p, p.seq_len - 4500, 61, 0, 40)


def test_units_without_a_key_tile():
    p = W.custom_prompt([("I", 38649), ("T", 7)], [D, D, S, S], 1, 128, dtype="bf16", span_sink=0, img_bidir=True,
                        name="shares-empty-rows")
    out = parity(p, 0, 62, bs.BS_MAP_REGROUP_ROWS, 30)
    assert not out[2:, :38649].any()   # nothing to see: zeros
