"""The decode kernel on a base weight kept in 4-bit groups (Sec. 5 "Model": the Q4_0 base of settings S2 and S3), with
bf16 pools and pools of 8-bit blocks, against the oracle on the same codes and scales, through the C-ABI.  Tolerance: one
bf16 rounding of y and one of every weight (2^-9 each) are far inside the layer's 1e-2."""
import numpy as np
import pytest
import torch

from gpu_harness import DeviceCase, rel_err, y_to_f64
from paper_2507_01438_amd import inputs as I

pytestmark = pytest.mark.gpu
DECODE = 1
TOL = 1e-2


def _case(seed, K, N, T, pool, ranks, q8=False, **kw):
    w = I.small_workload(seed, I.BF16, K, N, T, pool, ranks, wfmt=I.W_INT4_G32, **kw)
    return DeviceCase(w, w.projections[0], q8=q8)


# (K, N, T, pool, ranks): 1 to 4 blocks of 16 rows of x, one to eight K-slices per tile, a ragged last tile
SHAPES = [
    (256, 16, 1, 2, (8,)),
    (512, 80, 5, 3, (16, 8, 24)),
    (2048, 208, 20, 4, (16, 64, 8, 32)),
    (1024, 144, 33, 5, (8, 16, 32)),
    (4096, 256, 48, 4, (16,)),
    (2048, 528, 64, 6, (8, 16, 32, 64)),
    (4096, 4096, 32, 8, (16,)),
    (14336, 512, 64, 4, (8, 64)),
    (512, 32768, 64, 3, (8, 16)),          # 256 tiles of 128 rows, one K-slice each
]


@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_decode_kernel_reads_the_4bit_base(shape, q8):
    K, N, T, pool, ranks = shape
    case = _case(1500 + K + T, K, N, T, pool, ranks, q8, no_adapter_rows=(0,) if T > 1 else ())
    y = case.run()
    assert case.last_plan.path == DECODE and case.last_plan.n_launches == 1
    ref, base = case.reference(), case.base_reference()
    assert rel_err(y, ref) <= TOL
    assert np.max(np.max(np.abs(y - ref), axis=1) / np.max(np.abs(ref), axis=1)) <= 2e-2
    if np.max(np.abs(ref - base)) > 0:
        assert np.max(np.abs((y - base) - (ref - base))) / np.max(np.abs(ref - base)) <= 6e-2
    assert np.array_equal(y, case.run())          # fixed summation order
    assert case.pool.poll_error() == (0, -1)
    case.close()


@pytest.mark.parametrize("spin", [None, 0])
@pytest.mark.parametrize("shape", [(33, 256, 128, 3, (8, 16), (1, 32)), (64, 512, 192, 4, (8, 16, 32, 64), ()), (48, 1024, 1040, 5, (16,), (0,)),
                                   (64, 4096, 400, 6, (8, 24, 64), (63,)), (40, 512, 272, 4, (8, 20, 16, 3), (2,))])
def test_wide_decode_kernel_reads_the_4bit_base(shape, spin):
    from paper_2507_01438_amd import binding as B
    T, K, N, pool, ranks, none_rows = shape
    case = _case(1560 + T + N, K, N, T, pool, ranks, no_adapter_rows=none_rows)
    ref = case.reference()
    B.elora_debug_decode_wide(1)
    if spin is not None:
        B.elora_debug_spin_limit(spin)        # every wait runs out: the inputs, the 4-bit W among them, are read again
    try:
        y = case.run(force_path=DECODE)
        assert case.last_plan.path == DECODE and case.last_plan.tile_rows == 128
        y2 = case.run(force_path=DECODE)
    finally:
        B.elora_debug_decode_wide(-1)
        B.elora_debug_spin_limit(1 << 22)
    assert rel_err(y, ref) <= TOL and rel_err(y2, ref) <= TOL
    assert rel_err(case.run(force_path=DECODE), ref) <= TOL      # the same workspace serves the other kernel right after
    assert case.pool.poll_error() == (0, -1)
    case.close()


@pytest.mark.parametrize("T", [65, 130, 256])
def test_4bit_base_65_to_256_rows_in_passes(T):
    case = _case(1540 + T, 1024, 320, T, 6, (8, 16, 32))
    y = case.run()
    assert case.last_plan.path == DECODE and case.last_plan.n_launches == (T + 63) // 64
    assert rel_err(y, case.reference()) <= TOL
    case.close()


@pytest.mark.parametrize("T,K,Ns", [(20, 512, (4096, 1024)), (64, 2048, (144, 144, 1040)), (1, 256, (16, 32))])
def test_groups_of_calls_on_4bit_bases_run_as_one_launch(T, K, Ns):
    from paper_2507_01438_amd import binding as B
    cases = [_case(1570 + T, K, N, T, 6, ranks, no_adapter_rows=(T // 2,) if T > 1 else ()) for N, ranks in zip(Ns, [(16, 8, 32), (8,), (5, 64, 16)])]
    for _ in range(2):
        for c in cases:
            c.y.fill_(7)
        descs = B.desc_array([c.desc() for c in cases])
        assert B.elora_linear_group_launches(descs) == 1
        B.elora_batched_lora_linear_group(descs)
        torch.cuda.synchronize()
        for c in cases:
            assert rel_err(y_to_f64(c.y[: c.w.T], c.w.dtype), c.reference()) <= TOL, c.proj.N
            assert c.pool.poll_error() == (0, -1)
    for c in cases:     # one by one on the same workspaces: the mailboxes were left idle
        assert rel_err(c.run(), c.reference()) <= TOL
        c.close()
