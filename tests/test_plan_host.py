"""What a plan says of a call's launches (no GPU needed)."""
import pytest

from paper_2507_01438_amd import binding as B

FAKE = 0x7F0000000000


@pytest.mark.parametrize("T, K, N, launches, grid", [
    (8, 512, 512, 2, 32),                                     # 16 x 16 outputs per workgroup
    (100, 512, 512, 2, 4 * 32),                               # 32 x 16
    (1000, 512, 1000, 2, 32 * 32),                            # 32 x 32
    ((1 << 23) + 37, 1, 1024, 4, (1 << 23) - 1),              # more workgroups than a launch of fewer than 2^32 threads holds
    ((1 << 23) - 1, 1, 16, 2, 1 << 18),
    (1 << 23, 1, 16, 3, 1 << 18),                             # a row more than the shrink's launch holds
])
def test_fp32_plan(T, K, N, launches, grid):
    pool = B.elora_pool_create(K, N, 1, 2, B.ELORA_F32, FAKE, B.elora_pool_storage_bytes(K, N, 1, 2, B.ELORA_F32))
    d = B.make_desc(n_tokens=T, d_in=K, d_out=N, dtype=B.ELORA_F32, x=FAKE, W=FAKE, y=FAKE, workspace=FAKE, workspace_bytes=B.elora_workspace_bytes(T, K, N, 1),
                    pool=pool, adapter_idx=FAKE)
    p = B.elora_linear_plan(d)
    assert (p.path, p.n_launches, p.grid) == (B.ELORA_PATH_GENERIC, launches, grid)
    B.elora_pool_destroy(pool)
