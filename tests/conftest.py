import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run through the C-ABI on cuda:0)")


@pytest.fixture(params=[256, 128], ids=["tiles256", "band"])
def product(request):
    """Runs a test once on each matrix product of the GEMM path, whichever the rule would choose: the 256 x 256 tiles, and the
    tiles of a few hundred rows, 128 columns wide.  The value is a plan's tile_cols."""
    from paper_2507_01438_amd import binding as B
    B.elora_debug_band(0 if request.param == 256 else 1)
    yield request.param
    B.elora_debug_band(-1)
