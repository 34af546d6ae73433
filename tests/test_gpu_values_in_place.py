"""V tiles that are walked a few times are read where the caller has them, by transposing operand reads, those walked often come from a
transposed copy: prompts on both sides of the line, lengths around multiples of the 64-key tile, steps of one and of two tiles, both
entries, and a result that is written over V (where the copy has to stay)."""
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
from test_gpu_model import suffix_parity
from test_gpu_parity import full_parity
import workloads as W


@pytest.mark.skipif(shutil.which(bs_build.hipcc()) is None, reason="hipcc not available")
def test_kernels_that_transpose_have_no_mfma_hazard(monkeypatch):
    monkeypatch.setattr(isa_check, "KERNELS", ("_ZN2bs19attn_prefill_bf16_vILi128EEE", "_ZN2bs19attn_prefill_bf16_vILi64EEE",
                                               "_ZN2bs23attn_prefill_bf16_two_vILi64EEE"))
    res = isa_check.check()
    assert list(res.values()) == [[], [], []], res


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, bs.BS_MAP_PACK_KEYS])
@pytest.mark.parametrize("d,G,L", [(128, 2, 1537), (128, 2, 1600),             # steps per tile: some 6
                                   (128, 24, 1471), (128, 24, 1472), (128, 24, 1473),   # around 32
                                   (64, 1, 1665), (64, 1, 1600), (64, 1, 700),  # some 3, steps of two tiles and of one
                                   (64, 2, 1023), (64, 2, 1024), (64, 2, 1025), (64, 16, 1023)])   # from 4 on
def test_both_sides_of_the_line(d, G, L, flags):
    full_parity(prompt(L, 1, G, d), seed=81, flags=flags)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,window", [(70, 0), (300, 200), (700, 0), (1, 64)])
def test_chunks(rows, window, d):
    p = prompt(2111, 2, 2, d, **({"window": window} if window else {}))
    suffix_parity(p, p.seq_len - rows, 82, bs.BS_MAP_REGROUP_ROWS if window else bs.BS_MAP_PACK_KEYS, row_step=5)


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
