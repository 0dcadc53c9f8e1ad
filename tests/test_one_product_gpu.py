"""Calls of 65 to 256 rows as one matrix product: the shrink results reach the expand whole (24 bits), as in the decode kernel
that takes these calls too.  The adapters are made so that y shows every bit of them and nothing is rounded anywhere: rank
entries come in pairs whose results are 20-bit numbers that differ by a few units, B_i subtracts one from the other, W is
zero.  Every product and every sum, in whatever order, is a whole number of units below 2^24 of them, and y needs five bits:
the comparison is exact."""
import numpy as np
import pytest
import torch

from paper_2507_01438_amd import binding as B
from paper_2507_01438_amd import inputs as I

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GEMM = 2


def _bf16(a):
    return torch.from_numpy(I.f32_to_bf16_bits(np.ascontiguousarray(a, dtype=np.float32)).view(np.int16))


def _zero_w(K, N, wfmt):
    if wfmt == I.W_SAME:
        return torch.zeros((N, K), dtype=torch.int16, device=DEV), None
    scales = torch.ones((N, K // 32), dtype=torch.float16, device=DEV)
    if wfmt == I.W_INT8_G32:
        return torch.zeros((N, K), dtype=torch.int8, device=DEV), scales
    return torch.full((N, K // 2), 0x88, dtype=torch.uint8, device=DEV), scales


@pytest.mark.parametrize("wfmt", [I.W_SAME, I.W_INT8_G32, I.W_INT4_G32])
@pytest.mark.parametrize("K, N, T, lengths", [(2048, 2064, 200, None), (2048, 2064, 256, [100, 3, 0, 140, 13]), (4096, 1040, 80, [33, 47]), (1024, 36864, 200, [90, 110]),
                                              (1024, 36864, 256, None)])
def test_shrink_results_reach_the_expand_whole(K, N, T, lengths, wfmt):
    rng = np.random.default_rng(K + T)
    P, ranks = 5, (8, 16, 32, 64, 16)
    unit = 2.0 ** -7
    pool = B.AdapterPool(K, N, 64, P, B.ELORA_BF16)
    x = rng.integers(1, 4, size=(T, K)).astype(np.float64)
    keep = []
    for i in range(P):
        r = ranks[i]
        A = np.repeat(1.0 + unit * rng.integers(0, 128, size=(r // 2, K)), 2, axis=0)
        for p in range(r // 2):  # the second of a pair: a unit less in a few places
            at = rng.choice(np.flatnonzero(A[2 * p] > 1.0), size=8, replace=False)
            A[2 * p + 1, at] -= unit
        Bm = np.zeros((N, r))
        n = np.arange(N)
        sign = np.where(rng.integers(0, 2, size=N) == 1, 1.0, -1.0)
        Bm[n, 2 * (n % (r // 2))], Bm[n, 2 * (n % (r // 2)) + 1] = sign, -sign
        keep.append((A, Bm))
        pool.load(i, _bf16(A), _bf16(Bm), 2.0)
    torch.cuda.synchronize()
    n_req = T if lengths is None else len(lengths)
    who = rng.integers(-1, P, size=n_req).astype(np.int32)
    who[0] = 3
    rows = who if lengths is None else np.repeat(who, lengths)
    route = dict(adapter_idx=torch.from_numpy(who).to(DEV)) if lengths is None else dict(
        seg_offsets=torch.tensor([0] + np.cumsum(lengths).tolist(), dtype=torch.int32, device=DEV), seg_adapter=torch.from_numpy(who).to(DEV))
    W, w_scales = _zero_w(K, N, wfmt)
    lin = B.LoraLinear(K, N, B.ELORA_BF16, pool, T, DEV, wfmt=wfmt)
    xd, y = _bf16(x).to(DEV), torch.full((T, N), 7, dtype=torch.int16, device=DEV)
    over = (2.0 ** rng.integers(-2, 3, size=n_req)).astype(np.float32)
    for scales in (None, over):
        want = np.zeros((T, N))
        factor = np.full(n_req, 2.0) if scales is None else scales
        factor = factor if lengths is None else np.repeat(factor, lengths)
        for i, (A, Bm) in enumerate(keep):
            at = rows == i
            want[at] = factor[at, None] * ((x[at] @ A.T) @ Bm.T)
        assert np.abs(want).max() > 0
        d = lin.desc(xd, W, y, wfmt=wfmt, w_scales=w_scales, scales=None if scales is None else torch.from_numpy(scales).to(DEV), **route)
        plan = B.elora_linear_plan(d)
        assert plan.path == GEMM and plan.tile_cols == 128
        B.elora_batched_lora_linear(d)
        torch.cuda.synchronize()
        got = I.bf16_bits_to_f32(y.cpu().numpy().view(np.uint16)).astype(np.float64)
        np.testing.assert_array_equal(got, want)
    pool.close()


@pytest.mark.parametrize("scale", [1.5, np.inf])
@pytest.mark.parametrize("lengths", [None, [70, 1, 2, 100, 27]])
def test_an_infinite_entry_of_an_adapter_gives_an_infinity_of_its_sign(lengths, scale):
    """As a sum of fp32 products gives it: one infinite entry in a row of B_i makes that output infinite with the sign of the
    entry's shrink result; the other outputs, and the rows of other adapters, are as they were.  An infinite scale makes
    every output of its row infinite."""
    K = N = 2048
    T, P = 200, 4
    rng = np.random.default_rng(77)
    pool = B.AdapterPool(K, N, 32, P, B.ELORA_BF16)
    x = I.bf16_bits_to_f32(I.f32_to_bf16_bits(rng.standard_normal((T, K)).astype(np.float32))).astype(np.float64)
    keep = []
    for i, r in enumerate((8, 32, 24, 16)):
        A, Bm = [I.bf16_bits_to_f32(I.f32_to_bf16_bits(0.05 * rng.standard_normal(s).astype(np.float32))).astype(np.float64) for s in ((r, K), (N, r))]
        if i == 1:
            Bm[5, 9], Bm[700, 31], Bm[N - 1, 0] = np.inf, -np.inf, np.inf
        keep.append((A, Bm))
        pool.load(i, _bf16(A), _bf16(Bm), 1.0)
    torch.cuda.synchronize()
    n_req = T if lengths is None else len(lengths)
    who = (np.arange(n_req) % P).astype(np.int32)
    rows = who if lengths is None else np.repeat(who, lengths)
    route = dict(adapter_idx=torch.from_numpy(who).to(DEV)) if lengths is None else dict(
        seg_offsets=torch.tensor([0] + np.cumsum(lengths).tolist(), dtype=torch.int32, device=DEV), seg_adapter=torch.from_numpy(who).to(DEV))
    over = np.full(n_req, 1.5, dtype=np.float32)
    over[2] = scale
    row_scale = (over if lengths is None else np.repeat(over, lengths)).astype(np.float64)
    W, _ = _zero_w(K, N, I.W_SAME)
    lin = B.LoraLinear(K, N, B.ELORA_BF16, pool, T, DEV)
    xd, y = _bf16(x).to(DEV), torch.full((T, N), 7, dtype=torch.int16, device=DEV)
    d = lin.desc(xd, W, y, scales=torch.from_numpy(over).to(DEV), **route)
    assert B.elora_linear_plan(d).tile_cols == 128
    B.elora_batched_lora_linear(d)
    torch.cuda.synchronize()
    got = I.bf16_bits_to_f32(y.cpu().numpy().view(np.uint16)).astype(np.float64)
    want = np.zeros((T, N))
    for i, (A, Bm) in enumerate(keep):
        at = np.flatnonzero(rows == i)
        want[at] = row_scale[at, None] * ((x[at] @ A.T) @ Bm.T)
    assert not np.isnan(want).any() and (np.isinf(want).sum(axis=1)[rows == 1] >= 3).all()
    np.testing.assert_array_equal(np.isinf(got), np.isinf(want))
    inf = np.isinf(want)
    np.testing.assert_array_equal(got[inf], want[inf])
    got, want = got[~inf], want[~inf]
    # (one rounding of y, 2^-9; fp32 sums of cancelling products: 2^-20 of the largest)
    assert (np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 2.0 ** -18 * np.abs(want).max()).all()
    pool.close()


@pytest.mark.parametrize("T, K, N, ranks, lengths, q8", [
    (235, 256, 592, (128, 8), [235], False),
    (217, 256, 1040, (5, 16, 30), [100, 0, 1, 116], False),      # ranks that are no multiples of 8: gathered
    (130, 768, 272, (8, 24, 64), [64, 66], True),                # adapters in 8-bit blocks
    (65, 256, 16, (16,), [30, 35], True),
    (214, 512, 336, (64, 8, 32), None, False),                   # a row per adapter
    (256, 256, 48, (16, 8), None, False),
])
def test_4bit_w_with_a_short_d_in(T, K, N, ranks, lengths, q8):
    """Against the oracle and against the generic kernels, with scales given too; and by the decode kernel, which the same call
    takes when it is asked to."""
    from gpu_harness import DeviceCase, assert_close, rel_err
    w = I.small_workload(5600 + T, I.BF16, K, N, T, 6, ranks, segments=lengths, wfmt=I.W_INT4_G32, no_adapter_rows=() if lengths else (0, T - 1))
    case = DeviceCase(w, w.projections[0], q8=q8)
    y = case.run()
    assert (case.last_plan.path, case.last_plan.tile_cols) == (GEMM, 128)
    ref = case.reference()
    assert_close(y, ref, case.base_reference(), f"{T} rows")
    assert np.array_equal(y, case.run())
    assert rel_err(y, case.run(force_path=0)) <= 1e-2 and case.last_plan.path == 0
    B.elora_debug_decode_passes(1)
    try:
        d = case.run()
    finally:
        B.elora_debug_decode_passes(-1)
    if not q8 or max(ranks) <= 64:
        assert case.last_plan.path == 1
    assert rel_err(y, d) <= 1e-2
    n = T if lengths is None else len(lengths)
    over = np.linspace(0.25, 3.0, n).astype(np.float32)
    y = case.run(scales=torch.from_numpy(over).to(DEV))
    ref, base = case.reference(row_scale=over if lengths is None else np.repeat(over, lengths)), case.base_reference()
    assert rel_err(y, ref) <= 1e-2
    # (the adapter term alone: the rounding of y, 2^-9 of it, and that of the weights, as much again at most, are 2^-8 of the
    # largest y; where a scale makes the term small that is more than the 4 % of it which assert_close allows)
    lora = np.abs(ref - base).max()
    assert np.abs(y - ref).max() <= max(4e-2 * lora, 2.0 ** -8 * np.abs(ref).max())
    assert case.pool.poll_error() == (0, -1)
    case.close()
