"""The GEMM path's shrink at the sizes where it can go wrong: tiles where two or more runs meet, K-slices whose sums meet in
memory, ranks around its passes of 16, 32 and 64 columns, rows without adapter, runs around the length of 8 below which
rows are computed one by one; bf16 pools and pools of 8-bit blocks, against the oracle.  (The shrink results are rounded to
bf16 like every matrix-core operand: 2^-9 of the adapter term, far inside the layer's 1e-2.)"""
import numpy as np
import pytest

from gpu_harness import DeviceCase, assert_close
from paper_2507_01438_amd import inputs as I

pytestmark = pytest.mark.gpu
GEMM = 2

SHAPES = [
    # (K, pool, ranks, segment lengths, adapter-less segments)
    (64, 3, (8, 16), [32, 33, 7, 8, 20], ()),                       # one span of K: three of the four waves have none
    (576, 5, (8, 16, 24), [9, 7, 8, 8, 40, 3, 25], (2,)),           # runs of 7, 8 and 9; three runs in one tile
    (2048, 4, (32, 24), [300], ()),                                 # K-slices
    (4096, 4, (32, 8), [50, 14, 100, 1, 1, 1, 60], (5,)),           # K-slices, tiles with two runs, single rows
    (4160, 3, (64, 40), [70, 90, 129], ()),                         # 65 spans on four slices; ranks up to 64
    (2048, 3, (136, 72, 8), [40, 260], ()),                         # ranks above one pass
    (14336, 3, (16,), [45, 230], (0,)),
]


@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_shrink_shapes(shape, q8, product):
    K, pool, ranks, lengths, none = shape
    w = I.small_workload(1700 + K, I.BF16, K, 96, sum(lengths), pool, ranks, segments=lengths, no_adapter_rows=none)
    case = DeviceCase(w, w.projections[0], q8=q8)
    y = case.run(force_path=GEMM)
    assert case.last_plan.path == GEMM and case.last_plan.tile_cols == product
    assert_close(y, case.reference(), case.base_reference(), f"{shape}")
    assert np.array_equal(y, case.run(force_path=GEMM))     # fixed summation order, counters back at zero
    assert case.pool.poll_error() == (0, -1)
    case.close()


@pytest.mark.parametrize("K", [256, 4096])
def test_an_infinite_scale_makes_its_rows_infinite(K, product):
    """Everything is positive, so an infinite scale gives plus infinity in every output of its rows: entries past the rank are
    zero whatever the scale (rank 3 in steps of 8 and 64, rank 8 in a step of 16), in long and short runs, with K-slices
    and without."""
    import torch

    from gpu_harness import to_dev
    N, lengths, ranks = 264, [150, 5, 90, 20, 60], (3, 8, 16, 24)
    w = I.small_workload(1790 + K, I.BF16, K, N, sum(lengths), 4, ranks, segments=lengths)
    w.seg_adapter = np.array([0, 1, 2, 3, 1], dtype=np.int32)
    case = DeviceCase(w, w.projections[0])
    case.x_h &= 0x7FFF
    case.W_h &= 0x7FFF
    case.x.copy_(to_dev(case.x_h))
    case.W.copy_(to_dev(case.W_h))
    for i, (A, Bm, s) in list(case.adapters.items()):
        A, Bm = A & 0x7FFF, Bm & 0x7FFF
        case.adapters[i] = (A, Bm, s)
        case.pool.load(i, torch.from_numpy(A.view(np.int16)), torch.from_numpy(Bm.view(np.int16)), s)
    torch.cuda.synchronize()
    scales = np.array([np.inf, np.inf, 2.0, 0.5, np.inf], dtype=np.float32)
    y = case.run(scales=torch.from_numpy(scales).to("cuda:0"), force_path=GEMM)
    assert case.last_plan.tile_cols == product
    rows = np.repeat(scales, lengths)
    assert (y[np.isinf(rows)] == np.inf).all()
    rest = np.flatnonzero(np.isfinite(rows))
    ref = case.reference(row_scale=np.where(np.isfinite(rows), rows, 1.0).astype(np.float32))[rest]
    assert np.abs(y[rest] - ref).max() <= 1e-2 * np.abs(ref).max()
    case.close()


@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("T, K, ranks", [(511, 320, (8, 16, 64, 24)), (512, 320, (8, 16, 64, 24)), (777, 4096, (16,)), (1300, 192, (8, 136, 72))])
def test_many_rows_in_short_runs(T, K, ranks, q8, product):
    """Around the count from which they are a launch of their own; more pieces than workgroups, ranks of one to nine pieces of 16,
    rows without adapter, a long run among them, scales given; and the same batch by segments."""
    import torch

    from paper_2507_01438_amd import binding as B
    w = I.small_workload(1800 + T, I.BF16, K, 136, T, 9, ranks, no_adapter_rows=(0, 77, T - 1))
    w.adapter_idx[130:190] = 3
    case = DeviceCase(w, w.projections[0], q8=q8)
    over = np.linspace(0.25, 2.0, T).astype(np.float32)
    y = case.run(scales=torch.from_numpy(over).to("cuda:0"), force_path=GEMM)
    assert case.last_plan.tile_cols == product and case.last_plan.n_launches == (4 if T >= 512 else 3)
    assert_close(y, case.reference(row_scale=over), case.base_reference(), f"{T} rows")
    if product == 256:  # (the same shrink whichever way the rows are named; every product adds them in its own order)
        d = case.lin.desc(case.x[:T], case.W, case.y, seg_offsets=torch.arange(T + 1, dtype=torch.int32, device="cuda:0"), seg_adapter=case.adapter_idx,
                          scales=torch.from_numpy(over).to("cuda:0"))
        case.y.fill_(7)
        B.elora_force_path(GEMM)
        try:
            B.elora_batched_lora_linear(d)
        finally:
            B.elora_force_path(-1)
        torch.cuda.synchronize()
        from gpu_harness import y_to_f64
        assert np.array_equal(y_to_f64(case.y[:T], I.BF16), y)
    assert case.pool.poll_error() == (0, -1)
    case.close()


@pytest.mark.parametrize("pool_size", [40, 4])   # (more adapters than an eighth of the rows, and fewer)
@pytest.mark.parametrize("K", [64, 576, 2048, 2560, 4096, 4672, 9280])
def test_single_rows_over_lengths_and_ranks(K, pool_size, product):
    """Rows of one run each: d_in below, at and beside whole loads of a wave (512 elements), one and several turns of them,
    walks that begin in the middle; ranks around the four entries of a wave and the 16 of a workgroup."""
    w = I.small_workload(1900 + K, I.BF16, K, 72, 70, pool_size, (1, 3, 4, 5, 15, 16, 18, 64) if pool_size == 40 else (1, 4, 18, 64), no_adapter_rows=(0, 33))
    case = DeviceCase(w, w.projections[0])
    y = case.run(force_path=GEMM)
    assert case.last_plan.tile_cols == product
    assert_close(y, case.reference(), case.base_reference(), f"{K} {pool_size}")
    assert np.array_equal(y, case.run(force_path=GEMM))
    case.close()


@pytest.mark.parametrize("by_segments", [False, True])
@pytest.mark.parametrize("T", [70, 530])         # in the tiles' launch and in one of their own
@pytest.mark.parametrize("K", [4608, 9280, 14336])
def test_single_rows_do_not_depend_on_their_place(K, T, by_segments, product):
    """Rows with the same x and the same adapter have the same bits wherever in the batch they stand and however they are named.
    Products of 2^24 and -2^24 a few loads apart in one lane's sum make the order of its additions show: what is added between
    them is rounded to whole numbers."""
    import torch

    from gpu_harness import y_to_f64
    from paper_2507_01438_amd import binding as B
    N, ranks = 72, (16, 5)
    w = I.small_workload(1950 + K, I.BF16, K, N, T, 2, ranks)
    w.adapter_idx = (np.arange(T) % 2).astype(np.int32)
    case = DeviceCase(w, w.projections[0])
    rng = np.random.default_rng(K)
    x, As = rng.standard_normal(K), [rng.standard_normal((r, K)) for r in ranks]
    for k, v in ((512 * 2 + 3, 4096.0), (512 * 6 + 3, -4096.0)):
        x[k] = 4096.0
        for A in As:
            A[:, k] = v
    case.x.copy_(torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).to(case.x.device).expand(T, K))
    case.W.zero_()
    for i, A in enumerate(As):
        case.pool.load(i, torch.from_numpy(A).to(torch.bfloat16).view(torch.int16), torch.from_numpy(case.adapters[i][1].view(np.int16)), 1.0)
    torch.cuda.synchronize()
    route = dict(seg_offsets=torch.arange(T + 1, dtype=torch.int32, device="cuda:0"), seg_adapter=case.adapter_idx) if by_segments else dict(adapter_idx=case.adapter_idx)
    d = case.lin.desc(case.x[:T], case.W, case.y, **route)
    B.elora_debug_band(0 if product == 256 else 1, 0, 1)  # (one K-slice: a tile's slices take turns at the runs)
    B.elora_force_path(GEMM)
    try:
        B.elora_batched_lora_linear(d)
    finally:
        B.elora_force_path(-1)
    torch.cuda.synchronize()
    y = y_to_f64(case.y[:T], I.BF16)
    assert np.abs(y).max() > 1.0
    for first in (0, 1):
        assert (y[first::2] == y[first]).all()
    case.close()


@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("T, pool", [(300, 40), (330, 40), (530, 80)])   # (more adapters than an eighth of the rows, fewer, a launch of their own)
@pytest.mark.parametrize("K", [64, 1024, 4096, 8256])
def test_long_runs_among_rows_that_name_their_adapters(K, T, pool, q8, product):
    """Runs of 8 rows and more in a batch of which the host expects none: ranks of several passes through the rings of 32 entries
    and of 64, which a tile's two workgroups take in turn; one, two and three such runs in a tile, a run over three tiles, a
    run without adapter; with and without K-slices.  The shrink is the same when the rows are named by segments."""
    import torch

    from gpu_harness import y_to_f64
    from paper_2507_01438_amd import binding as B
    w = I.small_workload(1980 + K + T, I.BF16, K, 96, T, pool, (8, 64, 136, 40, 16), no_adapter_rows=(0, T - 1))
    idx = w.adapter_idx
    idx[10:90] = 1                                        # rank 64 over three tiles
    idx[96:108], idx[108:128] = 2, 6                      # ranks 136 and 64 in one tile
    idx[128:138], idx[138:148], idx[148:160] = 3, 12, 4   # ranks 40, 136 and 16
    idx[160:192] = 7                                      # a whole tile, rank 136
    idx[200:212] = -1
    case = DeviceCase(w, w.projections[0], q8=q8)
    y = case.run(force_path=GEMM)
    assert case.last_plan.tile_cols == product
    assert_close(y, case.reference(), case.base_reference(), f"{K} {T}")
    assert np.array_equal(y, case.run(force_path=GEMM))
    if product == 256:  # (every product adds the shrink results in its own order)
        d = case.lin.desc(case.x[:T], case.W, case.y, seg_offsets=torch.arange(T + 1, dtype=torch.int32, device="cuda:0"), seg_adapter=case.adapter_idx)
        case.y.fill_(7)
        B.elora_force_path(GEMM)
        try:
            B.elora_batched_lora_linear(d)
        finally:
            B.elora_force_path(-1)
        torch.cuda.synchronize()
        assert np.array_equal(y_to_f64(case.y[:T], I.BF16), y)
    assert case.pool.poll_error() == (0, -1)
    case.close()
