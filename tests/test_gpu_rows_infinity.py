"""Few-row kernel: an infinity among the values of a key that every row sees, of the last part, is that infinity in the results of its channel, however many
parts the keys are split into; lanes of the merge that have no part of their own look at the last one."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from gpu_util import assert_close, oracle_rows
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 3])
@pytest.mark.parametrize("d,parts", [(128, 1), (128, 3), (128, 16), (128, 63), (128, 64), (128, 65), (128, 100), (128, 129), (64, 16), (64, 127), (64, 129), (64, 257)])
def test_infinite_value_in_the_last_part(d, parts, rows):
    L, channel = 128 * parts - 5, 21
    p = W.custom_prompt([("T", L)], [0, 1, 2], 1, d, dtype="bf16", sink_len=0, name=f"rows-infinity-{parts}-d{d}-r{rows}")
    q, k, v = W.make_qkv(p, 91, DEV)
    at = np.arange(L - rows, L, dtype=np.int32)
    want = oracle_rows(p, q, k, v, at)
    v[0, L - rows - 1, channel], v[0, L - rows - 1, channel + 1] = float("inf"), float("-inf")
    qs = q[:, L - rows:].contiguous()
    out = torch.full_like(qs, -7.0)
    tm = bs.bs_build_tilemap(p.spans, L, p.head_class, p.sink_len, 128, 64, q_begin=L - rows)
    print(p.name, flush=True)
    bs.bs_attn_prefill(qs, k, v, out, tm, bs.BS_BF16, p.n_q_heads, p.gqa_group, d, p.scale, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    assert (got[:, :, channel] == np.inf).all() and (got[:, :, channel + 1] == -np.inf).all()
    got[:, :, channel:channel + 2] = want[:, :, channel:channel + 2]
    for h in range(p.n_q_heads):
        assert_close(got[h], want[h], "bf16", f"{p.name} head {h}")
