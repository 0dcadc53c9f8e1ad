"""What a workspace has to hold (no GPU needed): room for the sums of K-slices and for the other parts of the shrink results only
where some kernel of the call's rows, shape and dtype may use it."""
import ctypes

import pytest

from paper_2507_01438_amd import binding as B

FAKE = 0x7F0000000000


def _mail(N):  # counters, shrink results and mailboxes of the decode kernel: 2 KiB per column, by tiles of at most 128 columns
    return 4096 + 4 * 64 * 256 + 2048 * ((N + 127) // 128 * 128)


@pytest.mark.parametrize("K, N", [(4096, 4096), (4096, 1024), (4096, 14336), (14336, 4096), (512, 512), (2048, 272)])
@pytest.mark.parametrize("rank", [8, 64])
def test_up_to_64_rows_of_a_decode_shape_need_no_room_for_sums(K, N, rank):
    for T in (1, 32, 64):
        rows = 3 * 256 + T * 12 + max(T * rank * 4, T * 64 * 2) + 256
        assert B.elora_workspace_bytes(T, K, N, rank) <= _mail(N) + rows + 1024, T


@pytest.mark.parametrize("K, N", [(4096, 4096), (4096, 1024), (14336, 4096), (1000, 1430), (1088, 264), (64, 8), (512, 40)])
@pytest.mark.parametrize("wfmt", [B.ELORA_W_SAME, B.ELORA_W_INT8_G32, B.ELORA_W_INT4_G32])
@pytest.mark.parametrize("rank", [8, 64, 200])
def test_a_workspace_for_more_rows_holds_every_smaller_layout(K, N, wfmt, rank):
    sizes = [B.elora_workspace_bytes_w(t, K, N, rank, wfmt) for t in list(range(1, 1100)) + [2000, 4096, 8000, 8192, 16384, 40000]]
    assert all(a <= b for a, b in zip(sizes, sizes[1:]))


def test_fp32_calls_need_no_room_for_sums():
    K = N = 4096
    T = 100
    d = dict(n_tokens=T, d_in=K, d_out=N, x=FAKE, W=FAKE, y=FAKE, workspace=FAKE, workspace_bytes=_mail(N) + 16384)
    plan = B.elora_plan_t()
    assert B.lib.elora_linear_plan(ctypes.byref(B.make_desc(dtype=B.ELORA_F32, **d)), ctypes.byref(plan)) == B.ELORA_OK
    assert B.lib.elora_linear_plan(ctypes.byref(B.make_desc(dtype=B.ELORA_BF16, **d)), ctypes.byref(plan)) == B.ELORA_E_STORAGE
