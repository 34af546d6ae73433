"""Values that are not finite at keys that a row does not see: the few-row kernel multiplies the values of every key of the cache,
with a probability of zero where a row does not see it, and the results of that row must not show it."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from gpu_util import assert_close, oracle_rows
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu
D, S, I, IS = 0, 1, 2, 3
CLASSES = [D, S, I, IS, IS, I, S, D]
LONG = [("T", 9), ("I", 250), ("T", 5), ("I", 400), ("T", 3)]
SHORT = [("T", 9), ("I", 50), ("T", 5), ("I", 30), ("T", 3)]      # one part: no merge of several
IMAGE_LAST = LONG[:-1]


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("what", ["v", "k"])
@pytest.mark.parametrize("d,runs,rows,flags,window", [(128, LONG, 20, bs.BS_MAP_PACK_KEYS, 0), (64, LONG, 20, 0, 0), (128, LONG, 32, bs.BS_MAP_PACK_KEYS, 300),
                                                      (128, SHORT, 12, bs.BS_MAP_PACK_KEYS, 0), (64, SHORT, 12, bs.BS_MAP_PACK_KEYS, 0),
                                                      (128, IMAGE_LAST, 1, bs.BS_MAP_PACK_KEYS, 0), (128, IMAGE_LAST, 7, 0, 0)])
def test_keys_that_a_row_does_not_see(d, runs, rows, flags, window, what, bad):
    p = W.custom_prompt(runs, CLASSES, 2, d, dtype="bf16", sink_len=9, span_sink=3, window=window,
                        name=f"rows-nonfinite-d{d}-r{rows}-f{flags}-w{window}-{what}{bad}")
    q, k, v = W.make_qkv(p, 71, DEV)
    q_begin, kv, channel = p.seq_len - rows, 1, 37
    j = int(p.spans[0][0]) + 40 if not window else p.seq_len - 200     # a key of the first image (with a window, of the last)
    clean = oracle_rows(p, q, k, v, np.arange(q_begin, p.seq_len, dtype=np.int32))
    x = v.clone()
    x[kv, j] = 0.0                                                     # a row's result moves with the key's values iff it sees the key
    seen = (oracle_rows(p, q, k, x, np.arange(q_begin, p.seq_len, dtype=np.int32)) != clean).any(axis=2)
    if what == "v":
        v[kv, j, channel] = bad
    else:
        k[kv, j] = bad
    qs = q[:, q_begin:].contiguous()
    out = torch.full_like(qs, -7.0)
    tm = bs.bs_build_tilemap(p.spans, p.seq_len, p.head_class, p.sink_len, 128, 64, flags=flags, window=window, q_begin=q_begin)
    print(p.name, flush=True)
    bs.bs_attn_prefill(qs, k, v, out, tm, bs.BS_BF16, p.n_q_heads, p.gqa_group, p.head_dim, p.scale,
                       torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    assert not seen.all() and seen.any()
    assert not np.isfinite(got[seen][:, channel]).any()
    if what == "v":   # the other channels of a row that sees the key are as they were
        got[:, :, channel][seen] = clean[:, :, channel][seen]
    else:
        got[seen] = clean[seen]
    for h in range(p.n_q_heads):
        assert_close(got[h], clean[h], "bf16", f"{p.name} head {h} class {p.head_class[h]}")
