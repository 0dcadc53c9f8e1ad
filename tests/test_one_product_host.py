"""Which kernel calls of 65 to 256 rows take, from the plan alone (no GPU needed).  Such a call may leave the decode kernel,
whose shrink results are fp32, only for the product of band.hip, which keeps them whole: the 256 x 256 tiles multiply them
rounded to bf16.  However wide W is, these calls run on one of the two."""
import pytest

from paper_2507_01438_amd import binding as B

FAKE = 0x7F0000000000
DECODE, GEMM = 1, 2


def _plan(T, K, N, rank, wfmt=0, segments=None, pool_slots=4):
    pool = B.elora_pool_create(K, N, rank, pool_slots, B.ELORA_BF16, FAKE, B.elora_pool_storage_bytes(K, N, rank, pool_slots, B.ELORA_BF16))
    route = dict(adapter_idx=FAKE) if segments is None else dict(seg_offsets=FAKE, seg_adapter=FAKE, n_segments=segments)
    ws = B.elora_workspace_bytes_w(T, K, N, rank, wfmt)
    p = B.elora_linear_plan(B.make_desc(n_tokens=T, d_in=K, d_out=N, dtype=B.ELORA_BF16, wfmt=wfmt, x=FAKE, W=FAKE, y=FAKE, w_scales=FAKE if wfmt else None,
                                        workspace=FAKE, workspace_bytes=ws, pool=pool, **route))
    B.elora_pool_destroy(pool)
    return p


@pytest.mark.parametrize("wfmt", [B.ELORA_W_SAME, B.ELORA_W_INT8_G32, B.ELORA_W_INT4_G32])
@pytest.mark.parametrize("segments", [None, 1, 8])
@pytest.mark.parametrize("K, N", [(2048, 2048), (2048, 24576), (4096, 14336), (4096, 36864), (4096, 40960), (4096, 65536), (4096, 128256)])
def test_calls_of_65_to_256_rows_never_reach_the_256_x_256_tiles(K, N, segments, wfmt):
    for T in (65, 100, 129, 200, 240, 250, 256):
        for rank in (16, 32, 256):
            p = _plan(T, K, N, rank, wfmt, segments)
            assert p.path == DECODE or (p.path == GEMM and p.tile_cols == 128), (T, rank, p.path, p.tile_rows, p.tile_cols)


def test_without_the_product_of_band_they_stay_on_the_decode_kernel():
    B.elora_debug_band(0)
    try:
        for wfmt in (B.ELORA_W_SAME, B.ELORA_W_INT8_G32):
            assert _plan(200, 4096, 4096, 32, wfmt, 1).path == DECODE
    finally:
        B.elora_debug_band(-1)
    # a choice of the testing hook that no call fits (more K-slices than K has blocks): the decode kernel too, no refusal
    B.elora_debug_band(1, 1, 0)  # (256 rows take two row tiles at least)
    try:
        assert _plan(256, 4096, 4096, 32, B.ELORA_W_INT8_G32, 1).path == DECODE
    finally:
        B.elora_debug_band(-1)


@pytest.mark.parametrize("T, K, N, rank, segments, path", [
    (235, 256, 592, 128, 1, GEMM),       # launches of the decode kernel / one product: 357 / 23 us
    (217, 256, 7392, 32, 8, GEMM),       # 101 / 29
    (214, 256, 3408, 64, None, GEMM),    # 149 / 42
    (168, 1024, 11152, 16, 8, GEMM),     # 107 / 48
    (102, 3840, 144, 8, None, DECODE),   # 32 / 36
    (130, 1024, 320, 16, None, DECODE),
    (200, 4096, 4096, 16, 1, GEMM),
])
def test_a_4bit_w_of_65_to_256_rows(T, K, N, rank, segments, path):
    assert _plan(T, K, N, rank, B.ELORA_W_INT4_G32, segments).path == path
