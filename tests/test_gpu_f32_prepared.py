"""After bs_tilemap_prepare an fp32 call takes no device memory: the plan is on the device and the workspace is there, for either
head dimension."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from gpu_util import assert_close, oracle_rows
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
def test_prepared_fp32_call_takes_no_memory(d):
    runs = [("T", 30), ("I", 500), ("T", 9), ("I", 700), ("T", 40)]
    p = W.custom_prompt(runs, [0, 1, 2, 3, 0, 3, 2], 1, d, dtype="f32", sink_len=5, name=f"f32-prepared-d{d}")
    q, k, v = W.make_qkv(p, 91, DEV)
    out = torch.full_like(q, float("nan"))
    st = torch.cuda.current_stream().cuda_stream
    tm = bs.bs_build_tilemap(p.spans, p.seq_len, p.head_class, p.sink_len, 128, 64, flags=bs.BS_MAP_PACK_KEYS)
    for layer in range(2):
        classes = np.roll(p.head_class, layer)
        tm.rebind(classes)
        tm.prepare(bs.BS_F32, p.gqa_group, st)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        print(p.name, "layer", layer, flush=True)
        bs.bs_attn_prefill(q, k, v, out, tm, bs.BS_F32, p.n_q_heads, p.gqa_group, d, p.scale, st)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free
    rows = np.arange(0, p.seq_len, 7, dtype=np.int32)
    p.head_class[:] = classes
    want = oracle_rows(p, q, k, v, rows)
    for h in range(p.n_q_heads):
        assert_close(out[h, torch.from_numpy(rows).long()].cpu().numpy(), want[h], "f32", f"head {h}")
