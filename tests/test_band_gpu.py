"""The matrix product for a few hundred rows at the sizes where it can go wrong: every tile height, ragged rows and columns,
K of one block up to more blocks than the ring has stages, K-slices (and slices without a block's worth of ring), runs
that begin and end inside 16-row blocks, ranks around its steps of 32 entries and ranks that are no multiples of 8, rows
without adapter; bf16, 8-bit and 4-bit W, bf16 pools and pools of 8-bit blocks; against the oracle, at the tolerance of
the layer (matrix-core operands rounded to bf16, sums in fp32, one rounding of y)."""
import numpy as np
import pytest

from gpu_harness import DeviceCase, assert_close
from paper_2507_01438_amd import inputs as I

pytestmark = pytest.mark.gpu
GEMM = 2

SHAPES = [
    # (K, N, segment lengths, pool, ranks, adapter-less segments, row tiles, K-slices)
    (64, 8, [5], 2, (8,), (), 1, 1),                                     # one block, fewer rows than a fragment
    (128, 136, [33], 3, (16, 24), (), 1, 2),                             # one block per slice, a second tile of 8 columns
    (192, 264, [40, 1, 1, 1, 20], 5, (8, 40, 64), (2,), 1, 1),           # 63 rows of 64
    (512, 128, [16, 17, 15, 16, 30], 4, (32,), (), 1, 3),                # runs at and beside the 16-row cuts
    (640, 384, [100, 27], 3, (72, 136), (), 1, 2),                       # ranks of more than one step; 127 rows
    (704, 160, [1] * 150, 9, (8, 16, 32, 64), (3, 77), 1, 4),            # a decode batch, a run per row
    (1088, 256, [190, 2], 3, (3, 20, 33), (), 1, 1),                     # ranks that are no multiples of 8; 192 rows
    (2048, 512, [100, 124], 3, (16, 32), (), 1, 8),                      # the tallest tile, the most slices
    (832, 200, [60, 70, 95], 3, (24,), (1,), 2, 5),                      # one row more than the tallest tile; 13 blocks on 5 slices
    (2624, 1032, [389], 2, (32,), (), 2, 4),
    (576, 296, [64, 100, 300, 1, 1, 30], 6, (32, 64), (), 3, 3),
]


@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("wfmt", [I.W_SAME, I.W_INT8_G32, I.W_INT4_G32])
@pytest.mark.parametrize("shape", SHAPES)
def test_band_shapes(shape, wfmt, q8):
    from paper_2507_01438_amd import binding as B
    K, N, lengths, pool, ranks, none, tiles, slices = shape
    if q8 and any(r % 8 for r in ranks):
        pytest.skip("8-bit blocks hold ranks that are multiples of 8")
    if wfmt == I.W_INT8_G32 and sum(lengths) <= 256:
        lengths = lengths + [257 - sum(lengths)]  # (smaller batches on an 8-bit W do not take the path)
        tiles = 2
    w = I.small_workload(2900 + K, I.BF16, K, N, sum(lengths), pool, ranks, segments=lengths, no_adapter_rows=none, wfmt=wfmt)
    case = DeviceCase(w, w.projections[0], q8=q8)
    ref, base = case.reference(), case.base_reference()
    for t, s in ((tiles, slices), (tiles + 1, 1), (0, 0)):
        B.elora_debug_band(1, t, s)
        try:
            y = case.run(force_path=GEMM)
            again = case.run(force_path=GEMM)
        finally:
            B.elora_debug_band(-1)
        assert case.last_plan.path == GEMM
        assert_close(y, ref, base, f"{shape} {t} {s}")
        assert np.array_equal(y, again)  # fixed summation order, counters back at zero
    case.close()
