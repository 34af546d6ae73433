"""bf16 calls whose query rows of one head take more than 4 GiB: a row's offset needs 33 bits."""
import pytest
import torch

import paper_2507_09071_amd as bs
from test_gpu_model import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 64])
def test_query_rows_beyond_four_gibibytes(d):
    far, window, n = 2 ** 32 // (2 * d), 64, 300   # first row whose offset needs 33 bits
    L = far + n
    gen = torch.Generator(device=DEV)
    gen.manual_seed(95)
    q, k, v = (torch.zeros((1, L, d), dtype=torch.bfloat16, device=DEV) for _ in range(3))
    for t in (q, k, v):                            # the rows that are compared, and those that a wrapped offset would name
        for at in (0, far - n):
            t[:, at:at + 2 * n].normal_(generator=gen)
    out = torch.full_like(q, float("nan"))
    tm = bs.bs_build_tilemap([], L, [0], 0, 128, 64, window=window)
    print("L", L, "d", d, flush=True)
    bs.bs_attn_prefill(q, k, v, out, tm, bs.BS_BF16, 1, 1, d, d ** -0.5, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for first in (window, far - window):
        row = torch.arange(first, first + n if first == window else L, device=DEV)[:, None]
        pos = torch.arange(first - window, int(row[-1]) + 1, device=DEV)
        s = q[0, row[:, 0]].double() @ k[0, pos].double().t() * d ** -0.5
        s = torch.where((pos[None] <= row) & (pos[None] > row - window), s, float("-inf"))
        want = torch.softmax(s, dim=1) @ v[0, pos].double()
        err = (out[0, row[:, 0]].double() - want).norm() / want.norm()
        assert err < 5e-3, (first, float(err))     # the tolerance of bf16 results
