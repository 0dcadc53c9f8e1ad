"""The fp32 kernels at the sizes where they can go wrong: fewer rows than a tile, one more than a tile, K below and around a
turn of 16 and a round of 8 waves, rows whose length is no multiple of anything, odd ranks and ranks above one piece of 16,
rows without adapter, every tile form.  Against the fp64 oracle; sums of at most K products in fp32 differ from it by at
most (K + rank) * 2^-24 of the sum of the products' magnitudes, in practice by the square root of the count: 1e-5 of the
largest output is 20 times what the largest K here gives."""
import numpy as np
import pytest

from gpu_harness import DeviceCase, rel_err
from paper_2507_01438_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = [
    # (K, N, T, pool, ranks)
    (1, 1, 1, 1, (1,)),
    (3, 5, 2, 2, (1, 3)),
    (15, 17, 16, 3, (4, 7)),
    (16, 16, 17, 3, (8,)),
    (127, 31, 33, 4, (5, 16, 1)),
    (129, 33, 16, 4, (17, 33)),
    (512, 512, 8, 4, (8,)),
    (1000, 1430, 155, 8, (3, 5, 8, 16)),
    (1030, 2050, 140, 5, (40, 9)),       # 32 x 32 tiles, the last ones of 2 columns and 12 rows
    (2049, 700, 65, 4, (128, 3)),
    (4097, 48, 3, 2, (256,)),
]


@pytest.mark.parametrize("segments", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_fp32_shapes(shape, segments):
    K, N, T, pool, ranks = shape
    lengths = [T - T // 2, 0, T // 2] if segments else None
    w = I.small_workload(4100 + K, I.F32, K, N, T, pool, ranks, segments=lengths, no_adapter_rows=(1,) if T > 1 else ())
    case = DeviceCase(w, w.projections[0])
    y = case.run()
    assert rel_err(y, case.reference()) <= 1e-5
    assert np.array_equal(y, case.run())       # fixed summation order
    assert case.pool.poll_error() == (0, -1)
    case.close()


def test_more_rows_and_tiles_than_one_launch_holds():
    """2^23 rows are 2^32 threads of the shrink, and 2^33 outputs 2^32 of the product: both go out in pieces."""
    import torch

    from paper_2507_01438_amd import binding as B
    dev, T, N = "cuda:0", (1 << 23) + 37, 1024
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    x, W = [torch.randn(s, generator=gen, device=dev) for s in ((T, 1), (N, 1))]
    pool = B.AdapterPool(1, N, 1, 2, B.ELORA_F32)
    A, Bm = torch.randn((2, 1, 1), generator=gen, device=dev), torch.randn((2, N, 1), generator=gen, device=dev)
    for i in range(2):
        pool.load(i, A[i].contiguous(), Bm[i].contiguous(), 0.5)
    idx = (torch.arange(T, device=dev, dtype=torch.int32) % 3) - 1
    lin = B.LoraLinear(1, N, B.ELORA_F32, pool, T, dev)
    y = torch.full((T, N), 7.0, device=dev)
    d = lin.desc(x, W, y, adapter_idx=idx)
    assert B.elora_linear_plan(d).n_launches == 4
    B.elora_batched_lora_linear(d)
    torch.cuda.synchronize()
    for a in (0, (1 << 22) - 8, (1 << 23) - 4096, T - 2000):
        rows = slice(a, min(a + 6000, T))
        on = (idx[rows] >= 0).double()[:, None]
        which = idx[rows].clamp(min=0).long()
        want = x[rows].double() @ W.double().T + 0.5 * on * (x[rows].double() * A[which, 0].double()) * Bm[which, :, 0].double()
        assert (y[rows].double() - want).abs().max() <= 1e-6 * want.abs().max()
    assert not (y == 7.0).all(dim=1).any()
    assert pool.poll_error() == (0, -1)
    pool.close()


@pytest.mark.parametrize("shape", [(40, 8216, 5, 3, (1, 8)), (300, 9001, 16, 4, (3, 17, 24)), (33, 1000, 611, 4, (1, 5, 2)), (257, 515, 1025, 3, (9, 40))])
def test_fp32_launches_of_more_workgroups_than_fit_at_once(shape):
    """Many outputs: one turn's loads ahead, 16 x 16 and 32 x 32 tiles; K of fewer turns than waves, of one more than a round
    of the eight waves has, pools whose ranks need one to eight waves of the shrink."""
    K, N, T, pool, ranks = shape
    w = I.small_workload(4200 + K, I.F32, K, N, T, pool, ranks, no_adapter_rows=(1,))
    case = DeviceCase(w, w.projections[0])
    y = case.run()
    assert case.last_plan.grid > 512
    assert rel_err(y, case.reference()) <= 1e-5
    assert np.array_equal(y, case.run())
    assert case.pool.poll_error() == (0, -1)
    case.close()


@pytest.mark.parametrize("segments", [False, True])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1, (1,)), (15, 17, 2, 2, (3, 16)), (16, 16, 16, 2, (16,)), (63, 33, 17, 2, (16, 1)), (130, 40, 33, 4, (8, 5)), (512, 512, 8, 4, (8,)), (700, 35, 100, 1, (32,))])
def test_fp32_in_one_launch(shape, segments):
    """Calls whose rows meet at most 32 ranks: tiles of 16 rows and columns with and without a remainder, K below, at and
    behind a turn of 16 and a round of four waves, one and two blocks of ranks, rows without adapter and with a bad index."""
    K, N, T, pool, ranks = shape
    lengths = [T - T // 2, 0, T // 2] if segments else None
    w = I.small_workload(4300 + K, I.F32, K, N, T, pool, ranks, segments=lengths, no_adapter_rows=(1,) if T > 1 else ())
    case = DeviceCase(w, w.projections[0])
    y = case.run()
    assert case.last_plan.n_launches == 1
    assert rel_err(y, case.reference()) <= 1e-5
    assert np.array_equal(y, case.run())
    assert case.pool.poll_error() == (0, -1)
    if not segments and T > 2:
        case.adapter_idx[2] = pool + 3
        bad = case.run()
        ref = case.reference()
        ref[2] = case.base_reference()[2]
        assert rel_err(bad, ref) <= 1e-5
        assert case.pool.poll_error() == (1, 2)
    case.close()


def test_fp32_one_launch_captured_before_more_adapters_are_loaded():
    """A graph keeps its kernel: with ten more adapters in the pool its rows meet 11 of ranks 3 to 9, several walks over K."""
    import torch

    K, N, T, pool = 200, 50, 21, 12
    w = I.small_workload(4400, I.F32, K, N, T, pool, (9, 3, 8), no_adapter_rows=(4,))
    case = DeviceCase(w, w.projections[0], load_slots=[0])
    assert case.B.elora_linear_plan(case.desc()).n_launches == 1
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            case.B.elora_batched_lora_linear(case.desc(), stream)
    for i in range(1, pool):
        A, Bm, s = w.adapter(w.projections[0], i)
        case.adapters[i] = (A, Bm, s)
        case.pool.load(i, torch.from_numpy(A), torch.from_numpy(Bm), s)
    torch.cuda.synchronize()
    ref = case.reference()
    for _ in range(3):
        case.y.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert rel_err(case.y.cpu().numpy().astype(np.float64), ref) <= 1e-5
    assert case.pool.poll_error() == (0, -1)
    case.close()


@pytest.mark.parametrize("K, N, T, pool, ranks, launches", [
    (700, 64, 8, 2, (16,), 1), (701, 64, 8, 2, (16,), 2),                     # d_in
    (96, 8192, 16, 2, (8,), 1), (96, 8193, 16, 2, (8,), 2),                   # 512 tiles of 16 x 16, and 513
    (96, 4096, 17, 2, (8,), 1), (96, 4097, 17, 2, (8,), 2),                   # two rows of tiles
    (200, 64, 20, 4, (8,), 1), (200, 64, 20, 3, (11,), 2),                    # 32 ranks of the adapters there are, and 33
    (200, 64, 2, 9, (16,), 1), (200, 64, 3, 9, (16,), 2),                     # of the rows
])
def test_fp32_where_one_launch_ends(K, N, T, pool, ranks, launches):
    w = I.small_workload(4500 + K + N + T, I.F32, K, N, T, pool, ranks)
    case = DeviceCase(w, w.projections[0])
    y = case.run()
    assert case.last_plan.n_launches == launches
    assert rel_err(y, case.reference()) <= 1e-5
    case.close()
