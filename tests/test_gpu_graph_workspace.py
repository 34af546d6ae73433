"""Prepared calls in a captured graph whose partial results lie in the map's workspace: the replays stay right after eager calls of
the same map have taken a larger workspace and other maps have used what the library's block cache holds."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu


def inputs(hq, n_kv, L, rows, d, dtype):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(111)
    return [torch.empty((h, n, d), dtype=dtype, device=DEV).normal_(generator=gen) for h, n in ((hq, rows), (n_kv, L), (n_kv, L))]


def churn(stream):
    """Other maps of many sizes, each with a workspace of its own."""
    for L in (3000, 9000, 20000, 40000):
        q, k, v = inputs(8, 2, L, 300, 128, torch.bfloat16)
        out = torch.empty_like(q)
        tm = bs.bs_build_tilemap([(10, L - 50, 99)], L, np.arange(8) % 4, 5, 128, 64, q_begin=L - 300)
        bs.bs_attn_prefill(q, k, v, out, tm, bs.BS_BF16, 8, 4, 128, 128 ** -0.5, stream)
        tm.close()


@pytest.mark.parametrize("dtype,d,L,rows", [("bf16", 128, 48000, 517), ("f32", 64, 2000, 300), ("f32", 128, 2000, 300)])
def test_replays_after_the_workspace_grew(dtype, d, L, rows):
    n_kv, G = 4, 7
    hq, t = n_kv * G, torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = inputs(hq, n_kv, L, rows, d, t)
    want, out = torch.empty_like(q), torch.empty_like(q)
    tm = bs.bs_build_tilemap([(40, L // 2, 100), (L // 2 + 9, L - 40, 100)], L, np.arange(hq) % 4, 40, 128, 64, q_begin=L - rows)
    side = torch.cuda.Stream()

    def call(to):
        if dtype == "bf16":
            bs.bs_attn_prefill_static(q, k, v, to, tm, hq, G, d, d ** -0.5, side.cuda_stream)
        else:
            bs.bs_attn_prefill(q, k, v, to, tm, bs.BS_F32, hq, G, d, d ** -0.5, side.cuda_stream)

    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        tm.prepare(bs.BS_BF16 if dtype == "bf16" else bs.BS_F32, G, side.cuda_stream)
        call(want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    print(dtype, "d", d, "L", L, flush=True)
    with torch.cuda.graph(graph, stream=side):
        call(out)
    for replay in range(4):
        if replay == 1 and dtype == "bf16":   # the same binding: packed tiles and partial results of a plain call need more
            bs.bs_attn_prefill(q, k, v, out, tm, bs.BS_BF16, hq, G, d, d ** -0.5, side.cuda_stream)
        churn(side.cuda_stream)
        torch.cuda.synchronize()
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
            churn(side.cuda_stream)
        torch.cuda.synchronize()
        assert torch.isfinite(want.float()).all() and torch.equal(out, want), replay
