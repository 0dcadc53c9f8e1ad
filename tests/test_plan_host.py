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


@pytest.mark.parametrize("wfmt, T, n, launches", [
    (B.ELORA_W_SAME, 5000, 2, 2 + 2),
    (B.ELORA_W_SAME, 5000, 3, 2 + 3),
    (B.ELORA_W_INT8_G32, 5000, 2, 2 + 1 + 2),      # the copy of the second W is a launch of its own
    (B.ELORA_W_INT4_G32, 5000, 3, 2 + 2 + 3),
    (B.ELORA_W_INT4_G32, 400, 3, 2 + 3),           # no copy: the product takes W as it is stored
    (B.ELORA_W_INT8_G32, 300, 2, 2 + 2),
])
def test_launches_of_a_group_that_shares_its_shrink(wfmt, T, n, launches):
    K, N = 4096, 4096
    pools, descs = [], []
    for i in range(n):
        pools.append(B.elora_pool_create(K, N, 16, 4, B.ELORA_BF16, FAKE, B.elora_pool_storage_bytes(K, N, 16, 4, B.ELORA_BF16)))
        descs.append(B.make_desc(n_tokens=T, d_in=K, d_out=N, dtype=B.ELORA_BF16, wfmt=wfmt, x=FAKE, W=FAKE, y=FAKE + (i << 30), w_scales=FAKE if wfmt else None,
                                 workspace=FAKE + ((i + 1) << 36), workspace_bytes=B.elora_workspace_bytes_w(T, K, N, 16, wfmt), pool=pools[i], seg_offsets=FAKE, seg_adapter=FAKE, n_segments=2))
    assert all(B.elora_linear_plan(d).path == B.ELORA_PATH_GEMM and B.elora_linear_plan(d).n_launches == 3 for d in descs)
    assert B.elora_linear_group_launches(B.desc_array(descs)) == launches
    for p in pools:
        B.elora_pool_destroy(p)


@pytest.mark.parametrize("T, route, launches", [
    (600, dict(adapter_idx=FAKE), 4),                                                  # a row per adapter: their shrink is a launch of its own
    (500, dict(adapter_idx=FAKE), 3),
    (2168, dict(seg_offsets=FAKE, seg_adapter=FAKE, n_segments=124), 3),
    (2168, dict(seg_offsets=FAKE, seg_adapter=FAKE, n_segments=400), 4),
])
def test_launches_of_calls_with_many_short_runs(T, route, launches):
    K, N = 1024, 1024
    pool = B.elora_pool_create(K, N, 16, 4, B.ELORA_BF16, FAKE, B.elora_pool_storage_bytes(K, N, 16, 4, B.ELORA_BF16))
    descs = [B.make_desc(n_tokens=T, d_in=K, d_out=N, dtype=B.ELORA_BF16, x=FAKE, W=FAKE, y=FAKE + (i << 30), workspace=FAKE + ((i + 1) << 36),
                         workspace_bytes=B.elora_workspace_bytes(T, K, N, 16), pool=pool, **route) for i in range(2)]
    assert B.elora_linear_plan(descs[0]).n_launches == launches
    assert B.elora_linear_group_launches(B.desc_array(descs)) == launches + 1
    B.elora_pool_destroy(pool)


@pytest.mark.parametrize("T, K, N, wfmt, n_segments, tile_cols", [
    (2000, 1024, 1024, B.ELORA_W_SAME, None, 256),            # an adapter of up to 16 entries per row: 93 / 107 us on the two products
    (4000, 1024, 1024, B.ELORA_W_SAME, None, 256),            # 106 / 128
    (2000, 2752, 2896, B.ELORA_W_INT8_G32, 202, 256),         # two prompts and 200 rows of their own: 114 / 146
    (1200, 1024, 1024, B.ELORA_W_INT4_G32, 202, 256),         # 81 / 98
    (389, 4096, 14336, B.ELORA_W_SAME, 1, 128),               # a prompt: 121 / 73
    (1000, 4096, 4096, B.ELORA_W_SAME, 1, 128),               # 121 / 58
    (600, 4096, 4096, B.ELORA_W_SAME, None, 128),             # 185 / 103
])
def test_which_matrix_product_a_call_takes(T, K, N, wfmt, n_segments, tile_cols):
    pool = B.elora_pool_create(K, N, 16, 4, B.ELORA_BF16, FAKE, B.elora_pool_storage_bytes(K, N, 16, 4, B.ELORA_BF16))
    route = dict(adapter_idx=FAKE) if n_segments is None else dict(seg_offsets=FAKE, seg_adapter=FAKE, n_segments=n_segments)
    d = B.make_desc(n_tokens=T, d_in=K, d_out=N, dtype=B.ELORA_BF16, wfmt=wfmt, x=FAKE, W=FAKE, y=FAKE, w_scales=FAKE if wfmt else None, workspace=FAKE,
                    workspace_bytes=B.elora_workspace_bytes_w(T, K, N, 16, wfmt), pool=pool, **route)
    p = B.elora_linear_plan(d)
    assert (p.path, p.tile_cols) == (B.ELORA_PATH_GEMM, tile_cols)
    B.elora_pool_destroy(pool)
