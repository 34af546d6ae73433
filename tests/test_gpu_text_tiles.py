"""Compact tiles that only the kernels know: totals of text keys around multiples of the 64-key tile, windows, both kernels, chunks, and the
static entry where the tiles that a map publishes fit its scratch and those that the kernels know only with K read in place."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from test_gpu_model import suffix_parity
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
D, S, I, IS = 0, 1, 2, 3


def prompt(text, dtype, d, n_img=9, **kw):
    """`text` text tokens in front of, between and behind the images."""
    gaps = [text // (n_img + 1) + (i < text % (n_img + 1)) for i in range(n_img + 1)]
    runs = [("T", gaps[0])]
    for i in range(n_img):
        runs += [("I", [230, 333, 145][i % 3]), ("T", gaps[i + 1])]
    return W.custom_prompt(runs, [I, I, S, I, IS, D, I, IS], 2, d, dtype=dtype, sink_len=3, name=f"text{text}-{dtype}-d{d}",
                           value_recipe={"std": 1.0, "first_key_scale": 4.0}, **kw)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("text", [1, 63, 64, 65, 129])
def test_text_keys(text, dtype, d):
    p = prompt(text, dtype, d)
    tm = bs.bs_build_tilemap(p.spans, p.seq_len, p.head_class, p.sink_len, flags=bs.BS_MAP_PACK_KEYS)
    assert len(tm.walked(I, 0)[0]) == tm.n_k_tiles + -(-text // 64)
    full_parity(p, seed=91, flags=bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("rows", [150, 700])
def test_chunk(rows):
    p = prompt(65, "bf16", 128, img_bidir=True, sink_offsets=(0, 5, 64, 130))
    suffix_parity(p, p.seq_len - rows, 92, bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("window,bidir", [(64, False), (129, True), (700, False), (1500, True)])
def test_window(window, bidir, dtype, d):
    """Images of 256 with sinks all over them: compact tiles cut at both ends."""
    runs = [("T", 20)]
    for i in range(9):
        runs += [("I", 256), ("T", 12 + 5 * (i % 3))]
    p = W.custom_prompt(runs, [I, S, S, I, IS, D, IS, IS], 2, d, dtype=dtype, sink_len=3, name=f"window{window}-{bidir}-{dtype}",
                        span_sink=0, img_bidir=bidir, sink_offsets=tuple(range(3, 256, 13)), window=window,
                        value_recipe={"std": 1.0, "first_key_scale": 4.0})
    tm = bs.bs_build_tilemap(p.spans, p.seq_len, p.head_class, p.sink_len, flags=bs.BS_MAP_PACK_KEYS | (bs.BS_MAP_BIDIR_IMAGES if bidir else 0),
                             window=window, sink_offsets=p.sink_offsets)
    compact = sum(tm.walked(c, m)[2] for c in (S, I, IS) for m in range(tm.n_q_tiles))
    assert (compact > 0) == (window > 64)   # (images of more than twice the window keep the published lists)
    full_parity(p, seed=94, flags=bs.BS_MAP_PACK_KEYS)


def test_static_entry_with_more_tiles_than_published():
    hq, G, d, rows = 8, 1, 128, 300
    spans, pos = [], 30
    while len(spans) < 60:
        spans.append((pos, pos + 340, 8))
        pos += 340 + 30
    seq_len = 64 * 347 + 3
    assert spans[-1][1] < seq_len
    st = torch.cuda.current_stream().cuda_stream
    plain, static = (bs.bs_build_tilemap(spans, seq_len, [I] * 6 + [D, S], 5, flags=bs.BS_MAP_PACK_KEYS, q_begin=seq_len - rows)
                     for _ in range(2))
    known = len(static.walked(I, 0)[0])
    fits = bs.bs_static_scratch_bytes() // (hq * d * 256)
    assert static.n_k_tiles <= fits < known, (static.n_k_tiles, fits, known)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(93)
    q, k, v = (torch.empty((hq, n, d), dtype=torch.bfloat16, device="cuda:0").normal_(generator=gen) for n in (rows, seq_len, seq_len))
    want, got = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    print("static entry: tiles", static.n_k_tiles, known, flush=True)
    bs.bs_attn_prefill(q, k, v, want, plain, bs.BS_BF16, hq, G, d, d ** -0.5, st)
    static.prepare(bs.BS_BF16, G, st)
    bs.bs_attn_prefill_static(q, k, v, got, static, hq, G, d, d ** -0.5, st)
    torch.cuda.synchronize()
    assert torch.isfinite(want).all() and torch.equal(got, want)
