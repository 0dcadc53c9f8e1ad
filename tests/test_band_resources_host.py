"""The band and shrink kernels count their direct loads by hand too: no scratch memory (no GPU needed)."""
import os

import pytest

from test_kernel_resources_host import HIPCC, _scratch_of


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc here")
@pytest.mark.parametrize("source, kernel", [("band.hip", "lora_band_kernel"), ("shrink.hip", "sgmv_shrink_kernel")])
def test_no_scratch_memory(source, kernel):
    found = _scratch_of(source)
    assert any(kernel in k for k in found)
    assert all(v == 0 for v in found.values()), found
