"""An 8-bit base weight together with adapters kept in 8-bit blocks: the storage of the paper's setting S1 (Sec. 5
"Model": base model and adapters both in the block format the paper calls "Q8_0").  Decode kernel, decode group
launch, several passes, the wide kernel, waits that run out, and the GEMM path on the per-call bf16 copy; against the
oracle on the same codes and scales, through the C-ABI."""
import numpy as np
import pytest
import torch

from gpu_harness import DeviceCase, rel_err, y_to_f64
from paper_2507_01438_amd import inputs as I

pytestmark = pytest.mark.gpu
GENERIC, DECODE, GEMM = 0, 1, 2
TOL = 1e-2


def _case(seed, K, N, T, pool, ranks, **kw):
    w = I.small_workload(seed, I.BF16, K, N, T, pool, ranks, wfmt=I.W_INT8_G32, **kw)
    return DeviceCase(w, w.projections[0], q8=True)


# (K, N, T, pool, ranks): 1 to 4 blocks of 16 rows of x, one to eight K-slices per tile, a ragged last tile
SHAPES = [
    (256, 16, 1, 2, (8,)),
    (512, 80, 5, 3, (16, 8, 24)),
    (1024, 64, 16, 4, (8, 16)),
    (2048, 208, 20, 4, (16, 64, 8, 32)),
    (1024, 144, 33, 5, (8, 16, 32)),
    (4096, 256, 48, 4, (16,)),
    (2048, 528, 64, 6, (8, 16, 32, 64)),
    (4096, 4096, 32, 8, (16,)),
    (14336, 512, 64, 4, (8, 64)),
    (512, 32768, 64, 3, (8, 16)),          # 256 tiles of 128 rows, one K-slice each
]


@pytest.mark.parametrize("shape", SHAPES)
def test_decode_kernel_8bit_base_and_8bit_adapters(shape):
    K, N, T, pool, ranks = shape
    case = _case(1100 + K + T, K, N, T, pool, ranks, no_adapter_rows=(0,) if T > 1 else ())
    y = case.run()
    assert case.last_plan.path == DECODE and case.last_plan.n_launches == 1
    ref = case.reference()
    assert rel_err(y, ref) <= TOL
    base = case.base_reference()
    assert np.max(np.max(np.abs(y - ref), axis=1) / np.max(np.abs(ref), axis=1)) <= 2e-2
    if np.max(np.abs(ref - base)) > 0:
        assert np.max(np.abs((y - base) - (ref - base))) / np.max(np.abs(ref - base)) <= 6e-2
    assert np.array_equal(y, case.run())          # fixed summation order
    y_gen = case.run(force_path=GENERIC)          # a second reader of the same codes and scales
    assert case.last_plan.path == GENERIC
    assert rel_err(y, y_gen) <= TOL
    assert case.pool.poll_error() == (0, -1)
    case.close()


@pytest.mark.parametrize("spin", [None, 0])
@pytest.mark.parametrize("shape", [(33, 256, 128, 3, (8, 16), (1, 32)), (64, 512, 192, 4, (8, 16, 32, 64), ()),
                                   (48, 1024, 1040, 5, (16,), (0,)), (64, 4096, 400, 6, (8, 24, 64), (63,))])
def test_wide_decode_kernel_8bit_base_and_8bit_adapters(shape, spin):
    from paper_2507_01438_amd import binding as B
    T, K, N, pool, ranks, none_rows = shape
    case = _case(1130 + T + N, K, N, T, pool, ranks, no_adapter_rows=none_rows)
    ref = case.reference()
    B.elora_debug_decode_wide(1)
    if spin is not None:
        B.elora_debug_spin_limit(spin)       # every wait runs out at once: the fall-backs read both formats
    try:
        y = case.run(force_path=DECODE)
        assert case.last_plan.path == DECODE and case.last_plan.tile_rows == 128
        y2 = case.run(force_path=DECODE)
    finally:
        B.elora_debug_decode_wide(-1)
        B.elora_debug_spin_limit(1 << 22)
    assert rel_err(y, ref) <= TOL and rel_err(y2, ref) <= TOL
    assert rel_err(case.run(force_path=DECODE), ref) <= TOL      # the same workspace serves the 64-row kernel right after
    assert case.pool.poll_error() == (0, -1)
    case.close()


@pytest.mark.parametrize("T", [65, 130, 256])
def test_8bit_base_and_adapters_65_to_256_rows_in_passes(T):
    case = _case(1150 + T, 1024, 320, T, 6, (8, 16, 32))
    y = case.run()
    assert case.last_plan.path == DECODE and case.last_plan.n_launches == (T + 63) // 64
    assert rel_err(y, case.reference()) <= TOL
    case.close()


@pytest.mark.parametrize("T,K,Ns", [(40, 1024, (272, 64, 128)), (20, 512, (4096, 1024)), (64, 2048, (144, 144, 1040)),
                                    (64, 4096, (4096, 1024, 1024))])
def test_groups_on_8bit_bases_with_8bit_adapters_run_as_one_launch(T, K, Ns):
    from paper_2507_01438_amd import binding as B
    ranks_of = [(16, 8, 32), (8,), (8, 64, 16)][: len(Ns)]
    cases = []
    for N, ranks in zip(Ns, ranks_of):
        w = I.small_workload(1170 + T, I.BF16, K, N, T, 6, ranks, wfmt=I.W_INT8_G32, no_adapter_rows=(T // 2,) if T > 1 else ())
        cases.append(DeviceCase(w, w.projections[0], q8=True))
    for rep in range(2):
        for c in cases:
            c.y.fill_(7)
        descs = B.desc_array([c.desc() for c in cases])
        assert B.elora_linear_group_launches(descs) == 1
        B.elora_batched_lora_linear_group(descs)
        torch.cuda.synchronize()
        for c in cases:
            assert rel_err(y_to_f64(c.y[: c.w.T], c.w.dtype), c.reference()) <= TOL, (rep, c.proj.N)
            assert c.pool.poll_error() == (0, -1)
    for c in cases:
        c.close()


def test_many_rows_8bit_base_and_adapters_take_the_gemm_path(product):
    lengths = [300, 40, 1, 1, 280]
    w = I.small_workload(1190, I.BF16, 512, 264, sum(lengths), 4, (16, 8), wfmt=I.W_INT8_G32, segments=lengths)
    case = DeviceCase(w, w.projections[0], q8=True)
    y = case.run()
    assert case.last_plan.path == GEMM and case.last_plan.tile_cols == product
    assert rel_err(y, case.reference()) <= TOL
    case.close()


@pytest.mark.parametrize("names", [("q", "k", "v"), ("o",), ("gate", "up"), ("down",)])
def test_config3_layer_in_s1_storage_full_shapes(names):
    # the layer decode configuration with base and adapters both in 8-bit blocks, launched as the benchmark launches it
    from paper_2507_01438_amd import binding as B
    w = I.config3()
    w.wfmt = I.W_INT8_G32
    cases = [DeviceCase(w, I.LLAMA8B[n], load_slots=w.distinct_adapters(), q8=True) for n in names]
    descs = B.desc_array([c.desc() for c in cases])
    if len(cases) > 1:
        assert B.elora_linear_group_launches(descs) == 1
        B.elora_batched_lora_linear_group(descs)
    else:
        assert B.elora_linear_plan(cases[0].desc()).path == DECODE
        B.elora_batched_lora_linear(cases[0].desc())
    torch.cuda.synchronize()
    rng = np.random.default_rng(29)
    for c, n in zip(cases, names):
        cols = np.sort(rng.choice(c.proj.N, 48, replace=False))
        y = y_to_f64(c.y[: w.T], w.dtype)
        e = rel_err(y[:, cols], c.reference(cols=cols))
        print(f"config3, 8-bit base and adapters {names}: {n} rel err {e:.2e}")
        assert e <= TOL
        assert c.pool.poll_error() == (0, -1)
        c.close()
