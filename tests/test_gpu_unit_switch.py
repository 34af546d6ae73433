"""A workgroup of the bf16 kernel goes from unit to unit: the next one's record, query rows and first tiles are requested before the
present one is stored.  Lists of no, one, two, ... key tiles (more than three units a workgroup, so that the queues hand them out),
and nothing of a unit may reach the next."""
import numpy as np
import pytest
import torch

import paper_2507_09071_amd as bs
import workloads as W
from gpu_util import assert_close, oracle_rows, run_prefill

pytestmark = pytest.mark.gpu


def prompt(L, d, n_kv, G, sink=0):
    """Image first, no sinks unless asked for: rows of Sink heads see nothing (lists of no tile) up to the text at the end."""
    classes = np.random.default_rng([L, d]).integers(0, 4, n_kv * G)
    return W.custom_prompt([("I", L - 20), ("T", 20)], classes, n_kv, d, dtype="bf16", sink_len=0, span_sink=sink, name=f"switch-{L}-d{d}")


@pytest.mark.parametrize("flags", [0, bs.BS_MAP_PACK_KEYS])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [40, 84, 150, 212, 276, 340, 404])
def test_short_lists(L, d, flags):
    p = prompt(L, d, 260, 4, sink=0 if L < 200 else 7)
    q, k, v = W.make_qkv(p, 3, "cuda:0")
    got, tm = run_prefill(p, q, k, v, flags=flags)
    assert L < 150 or tm.pair_plan(4)["n_units"] > 3 * torch.cuda.get_device_properties(0).multi_processor_count
    heads = np.arange(0, p.n_q_heads, 4)[::5]
    heads = np.unique(np.concatenate([heads + i for i in range(4)]))   # whole groups: the oracle takes them as a prompt of its own
    part = W.custom_prompt([("I", L - 20), ("T", 20)], np.asarray(p.head_class)[heads], len(heads) // 4, d, dtype="bf16", sink_len=0,
                           span_sink=0 if L < 200 else 7, name="part")
    want = oracle_rows(part, q[heads], k[heads[::4] // 4], v[heads[::4] // 4])
    assert_close(got[heads].float().cpu().numpy(), want, "bf16", p.name)


@pytest.mark.parametrize("d", [64, 128])
def test_values_of_one_head_do_not_reach_the_others(d):
    p = prompt(404, d, 260, 4, sink=7)
    q, k, v = W.make_qkv(p, 3, "cuda:0")
    want, _ = run_prefill(p, q, k, v)
    v[::3] = float("nan")
    got, _ = run_prefill(p, q, k, v)
    clean = np.arange(p.n_q_heads) // 4 % 3 != 0
    assert torch.equal(got[clean], want[clean])
