"""fp32 calls whose keys lie more than 4 GiB into a KV head: compact tiles and the ragged last tile address single keys."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu
S, I, IS = 1, 2, 3


@pytest.mark.parametrize("d", [128, 64])
def test_keys_beyond_four_gibibytes(d):
    far = 2 ** 32 // (4 * d)                       # first key whose offset needs 33 bits
    text, image, L, rows = far - 100, far + 700, far + 700 + 1999, 100
    spans = [(0, text, 0), (image, L, 30)]         # an image without sinks, some text, the image the rows belong to
    k = torch.zeros((1, L, d), dtype=torch.float32, device=DEV)
    v = torch.zeros((1, L, d), dtype=torch.float32, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(95)
    k[:, text:].normal_(generator=gen)
    v[:, text:].normal_(generator=gen)
    q = torch.empty((3, rows, d), dtype=torch.float32, device=DEV).normal_(generator=gen)
    out = torch.full_like(q, float("nan"))
    tm = bs.bs_build_tilemap(spans, L, [S, I, IS], 0, 128, 64, flags=bs.BS_MAP_PACK_KEYS, q_begin=L - rows)
    print("L", L, "d", d, flush=True)
    bs.bs_attn_prefill(q, k, v, out, tm, bs.BS_F32, 3, 3, d, d ** -0.5, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    pos = torch.arange(text, L, device=DEV)
    kd, vd = k[0, text:].double(), v[0, text:].double()
    row = torch.arange(L - rows, L, device=DEV)[:, None]
    is_text, is_sink = pos < image, (pos >= image) & (pos < image + 30)
    for h, allowed in enumerate((is_text | is_sink, is_text | (pos >= image), is_text | (pos >= image))):
        s = q[h].double() @ kd.t() * d ** -0.5
        s = torch.where(allowed[None] & (pos[None] <= row), s, float("-inf"))
        want = torch.softmax(s, dim=1) @ vd
        err = (out[h].double() - want).norm() / want.norm()
        assert err < 3e-6, (h, float(err))         # fp32 sums of some 2,000 keys
