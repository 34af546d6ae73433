"""V tiles that are walked a few times are read where the caller has them, by transposing operand reads, those walked often come from a
transposed copy: prompts on both sides of the line, lengths around multiples of the 64-key tile, steps of one and of two tiles, units cut
and whole, both entries, and a result that is written over V (where the copy has to stay).  Which variant a case takes is asserted."""
import math
import shutil

import numpy as np
import pytest
import torch

import isa_check
import paper_2507_09071_amd as bs
from paper_2507_09071_amd import build as bs_build
from gpu_util import assert_close, oracle_rows
from test_gpu_keys_in_place import prompt
from launch_rules import variant
from test_gpu_model import suffix_parity
import workloads as W


@pytest.mark.skipif(shutil.which(bs_build.hipcc()) is None, reason="hipcc not available")
def test_kernels_that_transpose_have_no_mfma_hazard(monkeypatch):
    monkeypatch.setattr(isa_check, "KERNELS", ("_ZN2bs19attn_prefill_bf16_vILi128EEE", "_ZN2bs19attn_prefill_bf16_vILi64EEE",
                                               "_ZN2bs23attn_prefill_bf16_two_vILi64EEE"))
    res = isa_check.check()
    assert list(res.values()) == [[], [], []], res


N, R, P = 0, bs.BS_MAP_REGROUP_ROWS, bs.BS_MAP_PACK_KEYS
# head dimension, KV heads, group, tokens, rows (0: all), window, flags; two tiles a step, V transposed ahead, units cut
CASES = [
    # d = 128, up to 256 tiles (line at 22 steps a tile) ...
    (128, 1, 2, 1537, 0, 0, N, 0, 0, 1), (128, 1, 2, 1600, 0, 0, P, 0, 0, 1),
    (128, 1, 8, 1471, 0, 0, N, 0, 0, 1), (128, 1, 9, 1471, 0, 0, N, 0, 1, 1), (128, 1, 8, 1472, 0, 0, N, 0, 0, 1), (128, 1, 9, 1472, 0, 0, N, 0, 1, 1),
    (128, 1, 12, 1472, 0, 0, P, 0, 0, 1), (128, 1, 13, 1472, 0, 0, P, 0, 1, 1), (128, 1, 12, 1473, 0, 0, P, 0, 0, 1), (128, 1, 13, 1473, 0, 0, P, 0, 1, 1),
    # ... and more (32)
    (128, 12, 11, 1473, 0, 0, N, 0, 0, 0), (128, 12, 12, 1473, 0, 0, N, 0, 1, 0), (128, 12, 12, 1408, 0, 0, N, 0, 0, 0),
    (128, 10, 19, 1472, 0, 0, P, 0, 0, 0), (128, 10, 20, 1472, 0, 0, P, 0, 1, 0), (128, 10, 19, 1473, 0, 0, P, 0, 0, 0), (128, 10, 20, 1473, 0, 0, P, 0, 1, 0),
    # d = 64: up to 256 tiles always the copy
    (64, 8, 1, 1728, 0, 0, P, 0, 1, 1), (64, 8, 1, 1729, 0, 0, P, 0, 0, 1),
    # up to 4096 (line at 4)
    (64, 12, 1, 1601, 0, 0, N, 0, 0, 1), (64, 12, 2, 1601, 0, 0, N, 0, 1, 1), (64, 20, 2, 1025, 0, 0, P, 0, 0, 1), (64, 20, 2, 1601, 0, 0, P, 0, 1, 1),
    (64, 20, 2, 1024, 0, 0, P, 0, 0, 0), (64, 20, 1, 700, 0, 0, P, 0, 0, 0), (64, 20, 2, 1665, 0, 0, N, 1, 1, 0),
    (64, 8, 1, 16001, 300, 0, P, 0, 0, 1),
    (64, 8, 1, 16001, 300, 0, N, 1, 0, 1), (64, 8, 2, 16000, 300, 0, P, 1, 0, 1), (64, 8, 2, 16063, 300, 0, P, 1, 0, 1), (64, 8, 1, 16001, 600, 0, P, 1, 0, 1),
    (64, 8, 2, 16001, 500, 9000, R, 1, 0, 1),
    # and more (10), whole units
    (64, 66, 1, 4161, 0, 0, N, 1, 0, 0), (64, 64, 1, 4200, 0, 0, P, 1, 0, 0), (64, 64, 2, 4200, 0, 0, N, 1, 1, 0), (64, 64, 2, 4160, 0, 0, P, 1, 0, 0),
    (64, 64, 1, 4200, 0, 1500, R, 1, 0, 0), (64, 90, 2, 3001, 0, 1200, N, 1, 0, 0),
]


def build_map(p, rows, flags):
    return bs.bs_build_tilemap(p.spans, p.seq_len, p.head_class, p.sink_len, 128, 64, flags=flags, window=p.window, q_begin=p.seq_len - rows if rows else 0)


def assert_variant(tm, p, two, transposed, cut, n_wgs=256):
    v = variant(tm, p.head_class, p.n_kv_heads, p.head_dim, n_wgs)
    assert v[:2] == (bool(two), bool(transposed)) and bool(v[4]) == bool(cut), v


@pytest.mark.parametrize("d,n_kv,G,L,rows,window,flags,two,transposed,cut", CASES)
def test_cases_take_their_variants(d, n_kv, G, L, rows, window, flags, two, transposed, cut):
    p = prompt(L, n_kv, G, d, **({"window": window} if window else {}))
    assert_variant(build_map(p, rows, flags), p, two, transposed, cut)


@pytest.mark.gpu
@pytest.mark.parametrize("d,n_kv,G,L,rows,window,flags,two,transposed,cut", CASES)
def test_both_sides_of_the_line(d, n_kv, G, L, rows, window, flags, two, transposed, cut):
    p = prompt(L, n_kv, G, d, **({"window": window} if window else {}))
    q, k, v = W.make_qkv(p, 81, "cuda:0")
    begin = L - rows if rows else 0
    tm = build_map(p, rows, flags)
    assert_variant(tm, p, two, transposed, cut, torch.cuda.get_device_properties(0).multi_processor_count)
    print(p.name, n_kv, G, rows, window, flags, flush=True)
    qs = q[:, begin:].contiguous()
    out = torch.full_like(qs, float("nan"))
    bs.bs_attn_prefill(qs, k, v, out, tm, bs.BS_BF16, p.n_q_heads, G, d, p.scale, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out).all())
    some = np.unique(np.concatenate([np.arange(begin, L, 1 + (L - begin) * p.n_q_heads // 6000), np.arange(max(begin, L - 70), L, 3), [L - 1]])).astype(np.int32)
    got = out[:, torch.from_numpy(some - begin).long().to(out.device)].float().cpu().numpy()
    want = oracle_rows(p, q, k, v, some)
    for h in range(p.n_q_heads):
        assert_close(got[h], want[h], "bf16", f"{p.name} head {h} class {p.head_class[h]}")


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,window", [(70, 0), (300, 200), (700, 0), (1, 64)])
def test_chunks(rows, window, d):
    # (at d = 64 eight KV heads, so that the call has more than 256 tiles; in the short windows it has fewer, and takes the copy)
    p = prompt(2111, 8 if d == 64 else 2, 1 if d == 64 else 2, d, **({"window": window} if window else {}))
    flags = R if window else P
    v = variant(build_map(p, rows, flags), p.head_class, p.n_kv_heads, d)
    assert v[1] == (d == 64 and window > 0)
    suffix_parity(p, p.seq_len - rows, 82, flags, row_step=5)


@pytest.mark.gpu
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_result_over_the_values(d, static):
    p = prompt(777, 3, 1, d)
    q, k, v = W.make_qkv(p, 83, "cuda:0")
    want = oracle_rows(p, q, k, v)
    st = torch.cuda.current_stream().cuda_stream
    tm = bs.bs_build_tilemap(p.spans, p.seq_len, p.head_class, p.sink_len, 128, 64, flags=bs.BS_MAP_PACK_KEYS)
    if static:
        tm.prepare(bs.BS_BF16, 1, st)
        bs.bs_attn_prefill_static(q, k, v, v, tm, p.n_q_heads, 1, d, p.scale, st)
    else:
        bs.bs_attn_prefill(q, k, v, v, tm, bs.BS_BF16, p.n_q_heads, 1, d, p.scale, st)
    torch.cuda.synchronize()
    assert math.isfinite(float(v.float().abs().max()))
    assert_close(v.float().cpu().numpy().astype(np.float64), want, "bf16", "result over V")
