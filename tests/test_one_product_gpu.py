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
