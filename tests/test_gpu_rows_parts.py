"""Few-row kernel: the merge around the numbers of parts that it requests at once (64 and 128 at d = 128, 128 and 256 at d = 64; a
part holds 128 keys or more), with parts that a row sees nothing of, and waves of a part without a block."""
import numpy as np
import pytest

import paper_2507_09071_amd as bs
import workloads as W
from test_gpu_model import suffix_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 3])
@pytest.mark.parametrize("d,parts", [(128, 63), (128, 64), (128, 65), (128, 128), (128, 129), (64, 127), (64, 128), (64, 129), (64, 256), (64, 257)])
def test_parts_requested_at_once(d, parts, rows):
    L = 128 * parts - 97   # the last part: one block
    p = W.custom_prompt([("T", 9), ("I", L - 29), ("T", 20)], [0, 1, 2], 1, d, dtype="bf16", sink_len=9, name=f"rows-parts-{parts}-d{d}")
    suffix_parity(p, p.seq_len - rows, 49, bs.BS_MAP_PACK_KEYS)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("parts", [70, 140, 260])
def test_parts_that_a_row_sees_nothing_of(d, parts):
    # the last rows are an image's: the sparse heads' rows see no key of the long image in front of it
    L = 128 * parts
    p = W.custom_prompt([("T", 9), ("I", L - 49), ("T", 10), ("I", 30)], [0, 1, 2], 1, d, dtype="bf16", sink_len=9, name=f"rows-blind-{parts}-d{d}")
    suffix_parity(p, p.seq_len - 1, 50, bs.BS_MAP_PACK_KEYS)
