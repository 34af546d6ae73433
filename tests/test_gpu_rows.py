"""GPU parity of the few-row kernel (a decoding step, a handful of draft tokens) at the edges of its blocks: keys around
multiples of 32 and of four waves' share, one part and many, one and two row blocks and several row groups, both head
dimensions, text rows, image rows under sparse heads, windows and images that attend in both directions."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from test_gpu_model import DEV, suffix_parity

pytestmark = pytest.mark.gpu
D, S, I, IS = 0, 1, 2, 3


def prompt(L, classes, n_kv, d, **kw):
    """Text, images of up to 300 tokens and text between them, L tokens in all, ending with text."""
    runs, left = [("T", min(L, 7))], L - min(L, 7)
    while left > 60:
        n = min(300, left - 30)
        runs += [("I", n), ("T", min(20, left - n))]
        left -= n + min(20, left - n)
    runs.append(("T", left))
    return W.custom_prompt(runs, classes, n_kv, d, dtype="bf16", sink_len=min(3, L), name=f"rows-L{L}-d{d}-kv{n_kv}",
                           value_recipe={"std": 1.0, "first_key_scale": 4.0}, **kw)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [1, 31, 32, 33, 127, 128, 129, 1000, 4097])
def test_one_row(L, d):
    suffix_parity(prompt(L, [D, S, I, IS, S, D, I], 1, d), L - 1, 41, bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,n_kv,G", [(1, 3, 1), (2, 2, 7), (5, 2, 7), (13, 1, 5), (32, 1, 2), (31, 2, 7), (33, 2, 2)])
def test_row_counts(rows, n_kv, G, d):
    """Up to 32 rows of up to seven heads share a KV head; 33 rows go to the prefill kernel."""
    classes = np.arange(n_kv * G) % 4
    suffix_parity(prompt(1111, classes, n_kv, d), 1111 - rows, 42, bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("flags", [0, bs.BS_MAP_PACK_KEYS])
def test_image_rows_next_to_a_text_row(flags):
    """The last rows of an image and the text behind it under every class: masks of image rows are formed per key."""
    runs = [("T", 9), ("I", 250), ("T", 5), ("I", 400), ("T", 3)]
    p = W.custom_prompt(runs, [D, S, I, IS, IS, I, S, D], 2, 128, dtype="bf16", sink_len=9, name=f"rows-image-f{flags}")
    suffix_parity(p, p.seq_len - 20, 43, flags)


def test_image_rows_only():
    """Rows of an image only: the few-row kernel with a Dense head in the layer, the prefill kernel without one."""
    runs = [("T", 9), ("I", 250), ("T", 5), ("I", 400)]
    for classes in ([S, D, I, IS], [S, I, IS, IS]):
        p = W.custom_prompt(runs, classes, 2, 128, dtype="bf16", sink_len=9, name="rows-image-only")
        suffix_parity(p, p.seq_len - 7, 44, bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("window,bidir", [(1, False), (33, False), (700, False), (0, True), (150, True)])
def test_windows_and_bidirectional_images(window, bidir):
    runs = [("T", 20), ("I", 300), ("T", 9), ("I", 700), ("T", 4)]
    p = W.custom_prompt(runs, [S, I, IS, D, IS, S, I, D], 4, 128, dtype="bf16", sink_len=3, span_sink=0,
                        name=f"rows-window{window}-bidir{int(bidir)}", img_bidir=bidir, sink_offsets=(0, 5, 64, 130, 299, 650),
                        window=window)
    for rows in (1, 16):
        suffix_parity(p, p.seq_len - rows, 45, bs.BS_MAP_REGROUP_ROWS)


def test_static_call_and_streams_give_the_same_bits():
    p = prompt(3001, [D, S, I, IS, S, D, I], 1, 128)
    q, k, v = W.make_qkv(p, 46, DEV)
    qs = q[:, -2:].contiguous()
    tm = bs.bs_build_tilemap(p.spans, p.seq_len, p.head_class, p.sink_len, 128, 64, q_begin=p.seq_len - 2)
    args = (p.n_q_heads, p.gqa_group, p.head_dim, p.scale)
    want = torch.full_like(qs, float("nan"))
    bs.bs_attn_prefill(qs, k, v, want, tm, bs.BS_BF16, *args, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    other = torch.full_like(qs, float("nan"))
    bs.bs_attn_prefill(qs, k, v, other, tm, bs.BS_BF16, *args, side.cuda_stream)
    got = torch.full_like(qs, float("nan"))
    tm.prepare(bs.BS_BF16, p.gqa_group, torch.cuda.current_stream().cuda_stream)
    bs.bs_attn_prefill_static(qs, k, v, got, tm, *args, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(got, want) and torch.equal(other, want)
