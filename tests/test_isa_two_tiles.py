"""The hazard check of the compiled bf16 kernels, for the one whose steps take two key tiles."""
import shutil

import pytest

from paper_2507_09071_amd import build as bs_build
import isa_check


@pytest.mark.skipif(shutil.which(bs_build.hipcc()) is None, reason="hipcc not available")
def test_kernel_with_two_tiles_a_step_has_no_mfma_hazard(monkeypatch):
    monkeypatch.setattr(isa_check, "KERNELS", ("_ZN2bs21attn_prefill_bf16_twoILi64EEE",))
    res = isa_check.check()
    assert list(res.values()) == [[]], res
