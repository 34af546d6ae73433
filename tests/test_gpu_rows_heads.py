"""Few-row kernel with one row: head classes by 16-head words at every offset (an image row, so that the class counts), groups of
more than one and two row blocks, and more parts than the merge requests at once."""
import numpy as np
import pytest

import paper_2507_09071_amd as bs
import workloads as W
from test_gpu_model import suffix_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_kv,G", [(1, 1), (3, 11), (5, 7), (2, 33), (1, 70), (16, 2)])
def test_image_row_under_mixed_classes(n_kv, G, d):
    classes = np.random.default_rng([n_kv, G]).integers(0, 4, n_kv * G)
    classes[0] = 0   # a Dense head: without one the prefill kernel takes image rows
    p = W.custom_prompt([("T", 9), ("I", 250), ("T", 5), ("I", 401)], classes, n_kv, d, dtype="bf16", sink_len=9,
                        name=f"rows-heads-kv{n_kv}-g{G}-d{d}")
    suffix_parity(p, p.seq_len - 1, 47, bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("d,L", [(128, 33001), (64, 70003)])
def test_many_parts(d, L):
    p = W.custom_prompt([("T", 9), ("I", L - 29), ("T", 20)], [0, 1, 2], 1, d, dtype="bf16", sink_len=9, name=f"rows-parts-d{d}")
    suffix_parity(p, p.seq_len - 1, 48, bs.BS_MAP_PACK_KEYS)
