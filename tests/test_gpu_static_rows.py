"""Few query rows through the entry point that allocates nothing: the documented limit holds for them too, and a call of
bs_attn_prefill with the same binding prepares the map for it, as with any number of rows."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu


def inputs(hq, n_kv, L, rows, d, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return [torch.empty((h, n, d), dtype=torch.bfloat16, device=DEV).normal_(generator=gen) for h, n in ((hq, rows), (n_kv, L), (n_kv, L))]


@pytest.mark.parametrize("rows", [1, 32, 33])
def test_beyond_the_scratch_is_refused_for_any_number_of_rows(rows):
    n_kv, L, d = 8, 49216, 128           # 8 KV heads x 769 key tiles x 32 KB of packed tiles > 2 x 96 MiB
    q, k, v = inputs(n_kv, n_kv, L, rows, d, 101)
    out = torch.full_like(q, -7.0)
    st = torch.cuda.current_stream().cuda_stream
    tm = bs.bs_build_tilemap([(10, 2000, 0)], L, np.zeros(n_kv, np.uint8), 0, 128, 64, q_begin=L - rows)
    tm.prepare(bs.BS_BF16, 1, st)
    print("rows", rows, flush=True)
    with pytest.raises(bs.BlindsightError, match="static scratch") as e:
        bs.bs_attn_prefill_static(q, k, v, out, tm, n_kv, 1, d, d ** -0.5, st)
    assert e.value.code == -2
    torch.cuda.synchronize()
    assert bool((out == -7.0).all())     # nothing was launched


@pytest.mark.parametrize("rows,tail", [(1, 30), (20, 3), (32, 0), (40, 30)])
def test_a_plain_call_prepares_the_map(rows, tail):
    n_kv, G, L, d = 2, 4, 1500, 128
    q, k, v = inputs(n_kv * G, n_kv, L, rows, d, 102)
    want, got = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    st = torch.cuda.current_stream().cuda_stream
    classes = np.arange(n_kv * G) % 4
    tm = bs.bs_build_tilemap([(10, 700, 5), (705, L - tail, 9)], L, classes, 10, 128, 64, flags=bs.BS_MAP_PACK_KEYS, q_begin=L - rows)

    def static(group=G):
        bs.bs_attn_prefill_static(q, k, v, got, tm, n_kv * G, group, d, d ** -0.5, st)

    def refused(group=G):
        with pytest.raises(bs.BlindsightError) as e:
            static(group)
        assert e.value.code == -1

    print("rows", rows, "tail", tail, flush=True)
    refused()
    for layer in range(2):
        tm.rebind(np.roll(classes, layer))
        if layer:
            refused()                    # the binding of the first layer is stale
        bs.bs_attn_prefill(q, k, v, want, tm, bs.BS_BF16, n_kv * G, G, d, d ** -0.5, st)
        refused(2 * G)
        static()
        torch.cuda.synchronize()
        assert torch.isfinite(want).all() and torch.equal(got, want)
