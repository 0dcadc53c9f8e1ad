"""The band and shrink kernels count their direct loads by hand too: no scratch memory (no GPU needed)."""
import os
import re
import subprocess

import pytest

from test_kernel_resources_host import CSRC, HIPCC, _scratch_of


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc here")
@pytest.mark.parametrize("source, kernel", [("band.hip", "lora_band_kernel"), ("shrink.hip", "sgmv_shrink_kernel")])
def test_no_scratch_memory(source, kernel):
    found = _scratch_of(source)
    assert any(kernel in k for k in found)
    assert all(v == 0 for v in found.values()), found


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc here")
def test_two_workgroups_of_the_shrink_kernels_fit_by_their_registers():
    """A workgroup is a wave per SIMD: the single rows' own launch and the rings of up to 32 rank entries are sized for two per compute unit."""
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "--cuda-device-only", "-c", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wno-unused-command-line-argument", "-Rpass-analysis=kernel-resource-usage", "-o", os.devnull, os.path.join(CSRC, "shrink.hip")]
    p = subprocess.run(cmd, capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    waves = dict(zip(re.findall(r"Function Name: (\S+)", p.stderr), map(int, re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", p.stderr))))
    shrink = {k: v for k, v in waves.items() if "sgmv_shrink_kernel" in k or "shrink_rows_kernel" in k}
    assert len(shrink) == 8 and all(v >= 2 for v in shrink.values()), shrink
