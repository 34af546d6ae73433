"""bs_characterize_prompt packs K and V once for its four runs: the errors it reports are those of four separate calls, where all
runs take the few-row kernel, some of them do, units are cut (the workspace grows between runs) and queued."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from gpu_util import run_prefill

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("runs", [[("T", 7), ("I", 17)], [("I", 31)], [("T", 1), ("I", 32)], [("I", 300), ("T", 3), ("I", 410), ("T", 50)],
                                  [("T", 64), ("I", 1500), ("T", 9), ("I", 2100), ("T", 30)]])
def test_errors_are_those_of_separate_calls(runs, d):
    p = W.custom_prompt(runs, [0] * 6, 2, d, dtype="bf16", sink_len=3, span_sink=2, name="reuse")
    q, k, v = W.make_qkv(p, 61, "cuda:0")
    got_type, got = bs.bs_characterize_prompt(q, k, v, p.spans, p.seq_len, p.sink_len, bs.BS_BF16, p.n_q_heads, p.gqa_group, d,
                                              p.scale, 0.1, bs.BS_MAP_PACK_KEYS)
    outs = []
    for c in range(4):
        p.head_class[:] = c
        outs.append(run_prefill(p, q, k, v, flags=bs.BS_MAP_PACK_KEYS)[0].double())
    ref = (outs[0] ** 2).sum(dim=(1, 2))
    want = torch.stack([((o - outs[0]) ** 2).sum(dim=(1, 2)) / ref for o in outs[1:]]).cpu().numpy()
    # the same outputs to the bit; differences of bf16 values are formed in fp32 (2^-24 each), sums in fp64
    np.testing.assert_allclose(got, want, rtol=2.0 ** -22, atol=1e-300)
    passed = got < 0.1
    assert (got_type == np.where(passed[0], 1, np.where(passed[1], 2, np.where(passed[2], 3, 0)))).all()
