"""The entry point that allocates nothing gives the bits of the allocating one also where the packed tiles leave little of its
scratch and the launch cuts its units."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,rows,d,n_kv,G", [(48000, 517, 128, 4, 7), (40000, 300, 128, 4, 7), (95000, 1024, 64, 4, 4)])
def test_chunk_that_leaves_no_room_behind_the_packed_tiles(L, rows, d, n_kv, G):
    pos, spans = 40, []
    while pos < L - 3000:
        spans.append((pos, pos + 2500, 250))
        pos += 2530
    hq = n_kv * G
    tm, prepared = (bs.bs_build_tilemap(spans, L, np.arange(hq) % 4, 40, 128, 64, flags=bs.BS_MAP_REGROUP_ROWS, q_begin=L - rows)
                    for _ in range(2))
    assert tm.share_plan(G, torch.cuda.get_device_properties(0).multi_processor_count)["n_cut_units"] > 0
    gen = torch.Generator(device=DEV)
    gen.manual_seed(81)
    q, k, v = (torch.empty((h, n, d), dtype=torch.bfloat16, device=DEV).normal_(generator=gen) for h, n in ((hq, rows), (n_kv, L), (n_kv, L)))
    st = torch.cuda.current_stream().cuda_stream
    want, got = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    print("L", L, "rows", rows, "d", d, flush=True)
    bs.bs_attn_prefill(q, k, v, want, tm, bs.BS_BF16, hq, G, d, d ** -0.5, st)
    prepared.prepare(bs.BS_BF16, G, st)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    bs.bs_attn_prefill_static(q, k, v, got, prepared, hq, G, d, d ** -0.5, st)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
    assert torch.isfinite(want).all() and torch.equal(got, want)
