"""The matrix product for a few hundred rows at the sizes where it can go wrong: every tile height, ragged rows and columns,
K of one block up to more blocks than the ring has stages, K-slices (and slices without a block's worth of ring), runs
that begin and end inside 16-row blocks, ranks around its steps of 32 entries and ranks that are no multiples of 8, rows
without adapter; bf16, 8-bit and 4-bit W, bf16 pools and pools of 8-bit blocks; against the oracle, at the tolerance of
the layer (matrix-core operands rounded to bf16, sums in fp32, one rounding of y)."""
import numpy as np
import pytest

from gpu_harness import DeviceCase, assert_close, rel_err
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


@pytest.mark.parametrize("wfmt", [I.W_SAME, I.W_INT8_G32, I.W_INT4_G32])
@pytest.mark.parametrize("T, segments", [(129, False), (193, False), (256, True), (100, True)])
def test_65_to_256_rows_on_a_large_w_run_as_one_product(T, segments, wfmt):
    """No further from the oracle than the decode kernel, whose shrink results are fp32 (y is rounded to bf16 in both, which
    is nearly all of either's error; test_one_product_gpu.py has a comparison that shows every bit of them)."""
    import torch

    from paper_2507_01438_amd import binding as B
    lengths = ([T - 21, 0, 21] if T <= 128 else [T - 40, 0, 17, 1, 1, 21]) if segments else None
    w = I.small_workload(5100 + T, I.BF16, 2048, 2056 if wfmt == I.W_SAME else 2064, T, 9, (8, 16, 32, 64, 24), segments=lengths, wfmt=wfmt,
                         no_adapter_rows=(1,) if segments else (0, 64, T - 1))
    case = DeviceCase(w, w.projections[0])
    y = case.run()
    decode = T == 129 and wfmt != I.W_SAME     # (a row per adapter on a converted W: from 193 rows)
    assert case.last_plan.path == (1 if decode else GEMM) and case.last_plan.n_launches == 3
    ref = case.reference()
    assert_close(y, ref, case.base_reference(), f"{T} rows")
    assert np.array_equal(y, case.run())
    if w.projections[0].N % 16 == 0:
        d = case.run(force_path=1)
        assert case.last_plan.path == 1
        assert np.linalg.norm(y - ref) <= 1.005 * np.linalg.norm(d - ref)
    n = len(lengths) if segments else T
    over = np.linspace(0.25, 3.0, n).astype(np.float32)
    y = case.run(scales=torch.from_numpy(over).to("cuda:0"))
    rows = np.repeat(over, lengths) if segments else over
    assert_close(y, case.reference(row_scale=rows), case.base_reference(), f"{T} rows, scales given")
    assert case.pool.poll_error() == (0, -1)
    case.close()


def test_an_infinite_adapter_stays_in_its_own_rows():
    """A row takes nothing from another row's adapter, not even zero times its entries."""
    import torch

    from paper_2507_01438_amd import binding as B
    w = I.small_workload(5400, I.BF16, 512, 256, 40, 3, (16,), segments=[5, 3, 20, 12])
    w.seg_adapter = np.array([0, 1, 2, 0], dtype=np.int32)
    case = DeviceCase(w, w.projections[0])
    A, Bm, s = case.adapters[1]
    case.pool.load(1, torch.from_numpy(A.view(np.int16)), torch.from_numpy(np.full_like(Bm, 0x7F80).view(np.int16)), s)
    torch.cuda.synchronize()
    B.elora_debug_band(1)
    try:
        y = case.run(force_path=GEMM)
    finally:
        B.elora_debug_band(-1)
    rest = np.r_[0:5, 8:40]
    assert not np.isfinite(y[5:8]).any() and np.isfinite(y[rest]).all()
    assert rel_err(y[rest], case.reference(rows=rest)) <= 1e-2
    case.close()


@pytest.mark.parametrize("tiles, slices", [(2, 1), (2, 3), (3, 2), (4, 4), (7, 1)])
@pytest.mark.parametrize("lengths", [[345], [112, 112, 121], [5, 90, 20, 200, 30], [100, 9, 1, 1, 1, 1, 1, 231], [37, 300, 8]])
def test_few_runs_in_a_tile(lengths, tiles, slices):
    """Prompts: up to three runs in a wave's rows (and K-slice) go over all of its blocks, more of them step by step; runs that begin and end
    inside 16-row blocks, ranks on both sides of the 32 entries a pass takes, runs shared out over K-slices, one adapter full
    of infinities (its rows take nothing but infinities and NaN, all others nothing of them)."""
    import torch

    from paper_2507_01438_amd import binding as B
    T = sum(lengths)
    w = I.small_workload(5500 + T + len(lengths), I.BF16, 512, 200, T, 5, (8, 24, 32, 40, 64), segments=lengths, no_adapter_rows=(2,) if len(lengths) == 3 else ())
    case = DeviceCase(w, w.projections[0])
    B.elora_debug_band(1, tiles, slices)
    try:
        y = case.run(force_path=GEMM)
        assert np.array_equal(y, case.run(force_path=GEMM))
        assert_close(y, case.reference(), case.base_reference(), f"{lengths} {tiles} {slices}")
        i = int(w.seg_adapter[len(lengths) // 2])
        own = np.repeat(np.asarray(w.seg_adapter), lengths) == i
        if i >= 0 and not own.all():
            A, Bm, s = case.adapters[i]
            case.pool.load(i, torch.from_numpy(A.view(np.int16)), torch.from_numpy(np.full_like(Bm, 0x7F80).view(np.int16)), s)
            torch.cuda.synchronize()
            z = case.run(force_path=GEMM)
            assert not np.isfinite(z[own]).any() and np.array_equal(z[~own], y[~own])
    finally:
        B.elora_debug_band(-1)
    case.close()


@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("T, K, N, wfmt", [
    (320, 1024, 520, I.W_INT8_G32),      # the fewest rows; a ragged last column tile
    (401, 2048, 2048, I.W_INT8_G32),
    (1000, 1088, 1024, I.W_INT8_G32),
    (768, 1024, 1032, I.W_INT4_G32),
    (1001, 2048, 1024, I.W_INT4_G32),
])
def test_on_the_bf16_copy_of_w(T, K, N, wfmt, q8):
    """Calls of a 4- or 8-bit W whose product runs on these tiles from the call's bf16 copy: against the oracle, against the
    256 x 256 tiles on that copy and this kernel's own conversion (which multiply the same bf16 weights), alone and as a group
    whose second copy is a launch of its own, and without adapters."""
    import torch

    from gpu_harness import y_to_f64
    from paper_2507_01438_amd import binding as B
    w = I.small_workload(5700 + T + K, I.BF16, K, N, T, 4, (16, 8, 32), segments=[T - 140, 100, 0, 39, 1], wfmt=wfmt, no_adapter_rows=(3,))
    case = DeviceCase(w, w.projections[0], q8=q8)
    y = case.run()
    assert (case.last_plan.path, case.last_plan.tile_cols, case.last_plan.n_launches) == (GEMM, 128, 3)
    assert_close(y, case.reference(), case.base_reference(), f"{T} {K} {N}")
    assert np.array_equal(y, case.run())
    for mode in (0, 1):
        B.elora_debug_band(mode)
        try:
            other = case.run()
        finally:
            B.elora_debug_band(-1)
        assert case.last_plan.tile_cols == (256, 128)[mode]
        assert rel_err(y, other) <= 8e-3   # (sums of the same products in another order, y rounded to bf16 twice: 2 x 2^-9)
    twin = DeviceCase(w, w.projections[0], q8=q8, share=case)
    descs = B.desc_array([case.desc(), twin.desc()])
    assert B.elora_linear_group_launches(descs) == 2 + 1 + 2
    case.y.fill_(7)
    twin.y.fill_(7)
    B.elora_batched_lora_linear_group(descs)
    torch.cuda.synchronize()
    assert all(np.array_equal(y_to_f64(c.y[:T], I.BF16), y) for c in (case, twin))
    d = case.lin.desc(case.x[:T], case.W, case.y, wfmt=wfmt, w_scales=case.w_scales)
    d.pool = None
    assert (B.elora_linear_plan(d).tile_cols, B.elora_linear_plan(d).n_launches) == (128, 2)
    case.y.fill_(7)
    B.elora_batched_lora_linear(d)
    torch.cuda.synchronize()
    assert rel_err(y_to_f64(case.y[:T], I.BF16), case.base_reference()) <= 1e-2
    twin.close()
    case.close()


@pytest.mark.parametrize("ks", [1, 3])
@pytest.mark.parametrize("T, lengths", [(27, None), (59, [50, 9]), (91, None), (123, [123]), (155, [1, 154]), (187, None), (219, [100, 119]), (389, [150, 1, 238]), (389, None)])
@pytest.mark.parametrize("ranks, q8", [((5, 12, 36), False), ((5, 16, 36, 64), False), ((8, 40), True)], ids=["gathered", "both", "blocks"])
def test_adapters_that_are_gathered(ranks, q8, T, lengths, ks):
    """Pools whose rows of B_i are all gathered, which have an instance of their own, and pools where some are: every tile
    height, shrink results whole and rounded, with K-slices and without, waves with and without steps."""
    from paper_2507_01438_amd import binding as B
    w = I.small_workload(6200 + T, I.BF16, 832, 200, T, 6, ranks, segments=lengths, no_adapter_rows=(0,) if lengths is None else ())
    case = DeviceCase(w, w.projections[0], q8=q8)
    B.elora_debug_band(1, 0 if T > 224 else 1, ks)
    try:
        y = case.run(force_path=GEMM)
        again = case.run(force_path=GEMM)
    finally:
        B.elora_debug_band(-1)
    assert case.last_plan.tile_cols == 128 and case.last_plan.split_k == ks
    assert_close(y, case.reference(), case.base_reference(), f"{ranks} {T}")
    assert np.array_equal(y, again)
    assert case.pool.poll_error() == (0, -1)
    case.close()


def test_a_graph_captured_over_gathered_adapters_takes_others_loaded_later():
    import torch

    from gpu_harness import y_to_f64
    K, N, T = 832, 200, 389
    w = I.small_workload(6300, I.BF16, K, N, T, 3, (5, 12, 64), segments=[130, 9, 250])
    w.seg_adapter = np.array([0, 2, 1], dtype=np.int32)
    case = DeviceCase(w, w.projections[0], load_slots=[0, 1])
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            case.B.elora_batched_lora_linear(case.desc(), stream)
    assert case.B.elora_linear_plan(case.desc()).tile_cols == 128
    A, Bm, s = w.adapter(w.projections[0], 2)
    assert A.shape[0] == 64
    case.adapters[2] = (A, Bm, s)
    case.pool.load(2, torch.from_numpy(A.view(np.int16)), torch.from_numpy(Bm.view(np.int16)), s)
    torch.cuda.synchronize()
    ref, base = case.reference(), case.base_reference()
    for _ in range(3):
        case.y.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert_close(y_to_f64(case.y[:T], I.BF16), ref, base)
    assert case.pool.poll_error() == (0, -1)
    case.close()
