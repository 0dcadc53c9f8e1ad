"""Performance cases of the batched multi-adapter LoRA linear layer: what a serving program has it do.

A case is one batch going through some of a transformer layer's projections (`proj`, a text of launch units), each
unit a single call or a group call of projections that read the same activations:

    q, o        hidden -> hidden            up     hidden -> inter        down   inter -> hidden
    qkv         hidden -> hidden, kv, kv    gateup hidden -> inter twice

over `layers` layers with weights, pools and activations of their own (a decode step walks through a model's layers,
so its weights are cold).  The batch has `prompts` prompts of `prompt_rows` rows in all, each prompt a segment with one
adapter, and `decode_rows` rows that each name their own adapter.  With prompts it is routed by segments, without by
one index per row.  `plain` is the share of requests without an adapter.  `ranks` lists what an adapter's rank is drawn
from, `alpha` is the exponent of the adapters' popularity (0: uniform).  `base` is the storage of W ("same", "int8",
"int4": groups of 32 with fp16 scales), `adapters` that of the pool ("same" or "q8": 8-bit blocks of 32).  `override`
gives every request a scale of its own.  `universe` > 0 puts the adapter cache in front: that many adapters live in
pinned host memory as 8-bit blocks, `layers` counts consecutive batches on one layer, and every batch acquires its
adapters, loads the missing ones on a copy stream and runs.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2507_01438_amd import binding as B

DEV = "cuda:0"
WFMT = {"same": B.ELORA_W_SAME, "int4": B.ELORA_W_INT4_G32, "int8": B.ELORA_W_INT8_G32}


def _case(name=None, **kw):
    c = dict(dtype="bf16", base="same", adapters="same", hidden=4096, kv=1024, inter=14336, proj="q", layers=1, prompts=0,
             prompt_rows=0, decode_rows=0, pool=64, ranks="16", alpha=0.0, plain=0.0, override=False, universe=0)
    c.update(kw)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # The fp32 configuration: one small call, where launches and latency are all there is.
        _case("fp32_small", dtype="fp32", hidden=512, decode_rows=8, pool=4, ranks="8"),
        # fp32 at ragged sizes (no multiple of anything, odd ranks, base-only requests): a model kept in fp32 to check
        # an adapter, a few prompts and decode rows in one batch.
        _case("fp32_ragged", dtype="fp32", hidden=1000, inter=1430, proj="up down", prompts=3, prompt_rows=150, decode_rows=5,
              pool=8, ranks="3,5,8,16", plain=0.1),
        # One interactive request: a whole layer for a single row.
        _case("layer_1_row", proj="qkv o gateup down", decode_rows=1, pool=16),
        # A decode batch on one projection, 32 requests with power-law adapters, over eight layers.
        _case("q_32_rows", layers=8, decode_rows=32, alpha=1.1),
        # The decode step of a full batch: 64 rows, 256 adapters of mixed rank, all seven projections of a layer.
        _case("layer_64_rows", proj="qkv o gateup down", decode_rows=64, pool=256, ranks="8,16,32,64"),
        # The storage of the 8-bit serving setting: base and adapters in 8-bit blocks, rank 32, 20 requests.
        _case("layer_20_rows_8bit", proj="qkv o gateup down", base="int8", adapters="q8", decode_rows=20, pool=50, ranks="32", alpha=1.0),
        # The storage of the 4-bit serving settings: 4-bit base, rank-16 adapters, 20 requests.
        _case("layer_20_rows_4bit", proj="qkv o gateup down", base="int4", decode_rows=20, pool=50, alpha=1.0),
        # A large decode batch that does not fit one launch of 64 rows, some requests without adapter, scales overridden.
        _case("mlp_150_rows", proj="gateup down", decode_rows=150, pool=128, ranks="8,16,32,64", plain=0.1, override=True),
        # The prefill of one prompt of ordinary length through a layer (time to first token).
        _case("layer_one_prompt", proj="qkv o gateup down", prompts=1, prompt_rows=389, pool=32, ranks="32"),
        # Sixteen prompts at once (the largest): gate, up and down on bf16 weights.
        _case("mlp_16_prompts", proj="gateup down", prompts=16, prompt_rows=7871, pool=128, ranks="32"),
        # A mixed batch on a 4-bit base: four prompts of 512 rows and 120 decode rows, 1024 adapters.
        _case("mixed_4bit", proj="up", base="int4", prompts=4, prompt_rows=2048, decode_rows=120, pool=1024, alpha=1.0),
        # Decode behind the adapter cache: 512 adapters in pinned host memory, 64 blocks, the misses loaded as they come.
        _case("cached_32_rows", layers=8, decode_rows=32, pool=64, alpha=1.1, universe=512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fp32", "decode", "decode", "decode", "decode", "large", "large", "prefill", "prefill", "mixed", "cached"])
    ranks = rng.choice(["8", "16", "16", "32", "8,16,32,64", "64"])
    common = dict(pool=_log_int(rng, 4, 256), alpha=rng.choice([0.0, 0.5, 1.0, 1.1]), plain=rng.choice([0.0, 0.0, 0.1]),
                  override=rng.random() < 0.2)
    if kind == "fp32":
        prompts = rng.choice([0, 1, 3])
        return _case(dtype="fp32", hidden=_log_int(rng, 64, 2048), inter=_log_int(rng, 64, 3000), proj=rng.choice(["q", "up", "up down"]),
                     prompts=prompts, prompt_rows=_log_int(rng, 8, 256) if prompts else 0, decode_rows=rng.randint(1, 16),
                     **{**common, "pool": rng.randint(2, 16), "ranks": rng.choice(["8", "4,7", "1,5,16"])})
    hidden = rng.choice([1024, 2048, 2560, 3072, 4096, 4096, 5120])
    # (the rows of x that `down` reads are inter long: not always a multiple of the decode kernel's K step)
    shape = dict(hidden=hidden, kv=hidden // rng.choice([1, 4, 8]), inter=rng.choice([64, 128, 256, 256, 256]) * max(8, int(hidden * rng.uniform(2.5, 3.5)) // 256))
    base = rng.choice(["same", "same", "int8", "int4"])
    q8 = "q8" if rng.random() < 0.3 else "same"
    if kind == "cached":
        return _case(layers=4, decode_rows=rng.randint(4, 40), universe=rng.randint(80, 512), **{**shape, **common, "pool": rng.randint(40, 64), "ranks": rng.choice(["8", "16", "32"]),
                                                                                            "alpha": rng.choice([0.5, 1.0, 1.1])})
    more = dict(base=base, adapters=q8, ranks=ranks, **shape, **common)
    if kind == "decode":
        return _case(proj=rng.choice(["q", "qkv o", "gateup down", "qkv o gateup down"]), layers=2, decode_rows=_log_int(rng, 1, 64), **more)
    if kind == "large":
        return _case(proj=rng.choice(["q", "qkv o", "gateup down"]), decode_rows=rng.randint(65, 256), **more)
    if kind == "prefill":
        prompts = rng.randint(1, 8)
        return _case(proj=rng.choice(["qkv o", "gateup down"]), prompts=prompts, prompt_rows=max(_log_int(rng, 60, 4096), 8 * prompts), **more)
    prompts = rng.randint(1, 4)
    return _case(proj=rng.choice(["qkv o", "up", "gateup down"]), prompts=prompts, prompt_rows=_log_int(rng, 100, 2100), decode_rows=rng.randint(2, 120), **more)


# ---- what a case is made of ------------------------------------------------------------------------------------------


def _units(case):
    """[(input name, [(K, N), ...]), ...]: the calls of a layer; calls with the same input read the same activations."""
    h, kv, i = case["hidden"], case["kv"], case["inter"]
    kinds = {"q": ("h", [(h, h)]), "qkv": ("h", [(h, h), (h, kv), (h, kv)]), "o": ("a", [(h, h)]), "up": ("m", [(h, i)]),
             "gateup": ("m", [(h, i), (h, i)]), "down": ("f", [(i, h)])}
    return [kinds[u] for u in case["proj"].split()]


def _ranks(case):
    return [int(r) for r in case["ranks"].split(",")]


def _rows(case):
    return case["prompt_rows"] + case["decode_rows"]


def _normal(shape, std, dtype, gen):
    return torch.randn(shape, generator=gen, device=DEV, dtype=dtype) * std


def _grouped(w, levels):
    """Absmax quantisation in blocks of 32 consecutive values: (codes as float, fp16 scales)."""
    g = w.float().reshape(-1, 32)
    scale = (g.abs().amax(1) / levels).half()
    codes = torch.clamp(torch.round(g / torch.where(scale == 0, torch.ones_like(scale), scale).float()[:, None]), -levels - 1, levels)
    return codes, scale


def _weight(case, K, N, gen, dtype):
    w = _normal((N, K), 0.02, dtype, gen)
    if case["base"] == "same":
        return w, None
    if case["base"] == "int8":
        codes, scale = _grouped(w, 127)
        return codes.clamp(-127, 127).to(torch.int8).reshape(N, K), scale.reshape(N, K // 32)
    codes, scale = _grouped(w, 7)
    nib = (codes + 8).to(torch.uint8).reshape(N, K)
    return (nib[:, 0::2] | (nib[:, 1::2] << 4)).contiguous(), scale.reshape(N, K // 32)


def _q8(flat):
    """[n, values] -> 8-bit blocks of 32 along the values: (int8 codes, fp16 scales)."""
    codes, scale = _grouped(flat, 127)
    return codes.clamp(-127, 127).to(torch.int8).reshape(flat.shape), scale.reshape(flat.shape[0], -1)


def _popular(n, pool, alpha, gen_cpu):
    weight = torch.arange(1, pool + 1, dtype=torch.float64) ** (-alpha)
    return torch.randperm(pool, generator=gen_cpu)[torch.multinomial(weight, n, replacement=True, generator=gen_cpu)].to(torch.int32)


def _pool(case, K, N, ranks, gen, dtype):
    """A pool with every block filled.  Adapter i: A [r, K] and B [N, r] at the start of a row of the sources."""
    n, most, q8 = len(ranks), max(ranks), case["adapters"] == "q8"
    pool = B.AdapterPool(K, N, most, n, B.ELORA_F32 if case["dtype"] == "fp32" else B.ELORA_BF16, DEV, q8=q8)
    a, b = _normal((n, most * K), 0.02, dtype, gen), _normal((n, N * most), 0.02, dtype, gen)
    slots, scales = list(range(n)), [2.0] * n
    if q8:
        (ac, asc), (bc, bsc) = _q8(a), _q8(b)
        B.elora_pool_load_adapters_q8(pool.handle, slots, ranks, scales, list(ac), list(asc), list(bc), list(bsc))
    else:
        B.elora_pool_load_adapters(pool.handle, slots, ranks, scales, list(a), list(b))
    torch.cuda.synchronize()  # (the sources are let go here)
    return pool


def _requests(case, gen_cpu, pool):
    """(adapter per request, rows per request): the prompts first, then the decode rows."""
    prompts, decode = case["prompts"], case["decode_rows"]
    if case["alpha"] == 0.0 and prompts and prompts <= pool:  # prompts of different users
        adapters = torch.cat([torch.randperm(pool, generator=gen_cpu)[:prompts].to(torch.int32), _popular(decode, pool, 0.0, gen_cpu) if decode else torch.zeros(0, dtype=torch.int32)])
    else:
        adapters = _popular(prompts + decode, pool, case["alpha"], gen_cpu)
    if case["plain"]:
        adapters[torch.rand(adapters.shape, generator=gen_cpu) < case["plain"]] = -1
    lengths = []
    if prompts:
        # lengths spread evenly over a factor of sixteen, as those of prompts are, adding up to prompt_rows
        share = torch.rand(prompts, generator=gen_cpu, dtype=torch.float64) * 15 + 1
        ends = torch.round(torch.cumsum(share, 0) / share.sum() * case["prompt_rows"]).to(torch.int64)
        lengths = [int(e - s) for s, e in zip([0] + ends.tolist()[:-1], ends.tolist())]
    return adapters, lengths + [1] * decode


class _State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    gen_cpu = torch.Generator()
    gen_cpu.manual_seed(seed)
    if case["universe"]:
        return _prepare_cached(case, gen, gen_cpu)
    s = _State()
    dtype, code = (torch.float32, B.ELORA_F32) if case["dtype"] == "fp32" else (torch.bfloat16, B.ELORA_BF16)
    rows, choices = _rows(case), _ranks(case)
    ranks = [choices[i] for i in torch.randint(len(choices), (case["pool"],), generator=gen_cpu).tolist()]
    adapters, lengths = _requests(case, gen_cpu, case["pool"])
    route = {}
    if case["prompts"]:
        route["seg_offsets"] = torch.tensor([0] + np.cumsum(lengths).tolist(), dtype=torch.int32, device=DEV)
        route["seg_adapter"] = adapters.to(DEV)
    else:
        route["adapter_idx"] = adapters.to(DEV)
    if case["override"]:
        route["scales"] = torch.rand(adapters.shape, generator=gen_cpu).add(0.5).to(DEV)
    s.calls, s.keep, s.outputs, s.parts = [], [route], [], []
    for _ in range(case["layers"]):
        inputs = {}
        for name, shapes in _units(case):
            K = shapes[0][0]
            if name not in inputs:
                inputs[name] = _normal((rows, K), 1.0, dtype, gen)
            x, descs = inputs[name], []
            for K, N in shapes:
                W, w_scales = _weight(case, K, N, gen, dtype)
                pool = _pool(case, K, N, ranks, gen, dtype)
                lin = B.LoraLinear(K, N, code, pool, rows, DEV, wfmt=WFMT[case["base"]])
                y = torch.zeros((rows, N), dtype=dtype, device=DEV)
                descs.append(lin.desc(x, W, y, wfmt=WFMT[case["base"]], w_scales=w_scales, **route))
                s.keep += [W, w_scales, pool, lin, x]
                s.outputs.append(y)
            s.calls.append(B.desc_array(descs) if len(descs) > 1 else descs[0])
    torch.cuda.synchronize()
    return s


def run(s):
    if hasattr(s, "cache"):
        return _run_cached(s)
    for call in s.calls:
        if isinstance(call, ctypes.Array):
            B.elora_batched_lora_linear_group(call)
        else:
            B.elora_batched_lora_linear(call)
    return s.outputs


# ---- decode behind the adapter cache -----------------------------------------------------------------------------------

RING = 64  # index uploads that may be under way


class _CachedState(_State):
    def __del__(self):
        torch.cuda.synchronize()
        B.elora_cache_destroy(self.cache)


def _pinned(t):
    host = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    host.copy_(t)
    return host


def _prepare_cached(case, gen, gen_cpu):
    s = _CachedState()
    K = N = case["hidden"]
    rank, rows, n, batches = _ranks(case)[0], _rows(case), case["universe"], case["layers"]
    s.cache = B.elora_cache_create(case["pool"])
    s.pool = B.AdapterPool(K, N, rank, case["pool"], B.ELORA_BF16, DEV)
    s.sources = [_pinned(t) for m in (rank * K, N * rank) for t in _q8(_normal((n, m), 0.02, torch.bfloat16, gen))]
    s.addresses = [[row.data_ptr() for row in t] for t in s.sources]
    s.rank, s.rows = rank, rows
    s.lin = B.LoraLinear(K, N, B.ELORA_BF16, s.pool, rows, DEV)
    s.W = _normal((N, K), 0.02, torch.bfloat16, gen)
    s.x = [_normal((rows, K), 1.0, torch.bfloat16, gen) for _ in range(batches)]
    s.outputs = [torch.zeros((rows, N), dtype=torch.bfloat16, device=DEV) for _ in range(batches)]
    s.ids = [_popular(rows, n, case["alpha"], gen_cpu).numpy() for _ in range(batches)]
    s.idx = torch.zeros((RING, rows), dtype=torch.int32, device=DEV)
    s.idx_host = torch.zeros((RING, rows), dtype=torch.int32, pin_memory=True)
    s.idx_np = s.idx_host.numpy()
    s.idx_free, s.at = [None] * RING, 0
    s.descs = [[s.lin.desc(s.x[b], s.W, s.outputs[b], adapter_idx=s.idx[r]) for r in range(RING)] for b in range(batches)]
    s.miss_ids, s.miss_slots = np.zeros(rows, np.int32), np.zeros(rows, np.int32)
    s.copy = torch.cuda.Stream()
    torch.cuda.synchronize()
    return s


def _run_cached(s):
    for b, ids in enumerate(s.ids):
        r = s.at % RING
        s.at += 1
        if s.idx_free[r] is not None:
            s.idx_free[r].synchronize()  # the upload that used this piece of pinned memory a ring ago
        else:
            s.idx_free[r] = torch.cuda.Event()
        slots = s.idx_np[r]
        n = B.elora_cache_acquire_batch(s.cache, ids, slots, s.miss_ids, s.miss_slots)
        if n:
            where, who = s.miss_slots[:n].tolist(), s.miss_ids[:n].tolist()
            B.elora_cache_load_begin(s.cache, where, s.copy)
            B.elora_pool_load_adapters_q8(s.pool.handle, where, [s.rank] * n, [2.0] * n, *[[a[i] for i in who] for a in s.addresses], s.copy)
            B.elora_cache_load_end(s.cache, where, s.copy)
        used = slots.tolist()
        B.elora_cache_batch_begin(s.cache, used)
        s.idx[r].copy_(s.idx_host[r], non_blocking=True)
        s.idx_free[r].record()
        B.elora_batched_lora_linear(s.descs[b][r])
        B.elora_cache_batch_end(s.cache, used)
        B.elora_cache_release_batch(s.cache, ids)
    return s.outputs


# ---- the least a pass can do ---------------------------------------------------------------------------------------------


def _distinct(draws, pool, alpha):
    """Expected number of different adapters among `draws` requests."""
    p = np.arange(1, pool + 1, dtype=np.float64) ** (-alpha)
    p /= p.sum()
    return float((1 - (1 - p) ** draws).sum())


def work(case):
    e = 4 if case["dtype"] == "fp32" else 2
    wb = {"same": e, "int8": 1 + 2 / 32, "int4": 0.5 + 2 / 32}[case["base"]]
    ab = 17 / 16 if case["adapters"] == "q8" else e
    rows, ranks = _rows(case), _ranks(case)
    rank = sum(ranks) / len(ranks)
    served = 1 - case["plain"]
    if case["universe"]:
        # W, x and y per batch, the distinct adapters of the pass's requests, and over the bus those that a cache of this
        # size cannot keep from one pass to the next
        K = N = case["hidden"]
        each = _distinct(rows, case["universe"], case["alpha"]) * rank * (K + N) * e
        total = _distinct(rows * case["layers"], case["universe"], case["alpha"])
        missing = max(0.0, total - case["pool"]) * rank * (K + N) * 17 / 16
        return {"bytes": case["layers"] * (N * K * e + rows * (K + N) * e + each) + missing,
                "flops": case["layers"] * (2 * rows * K * N + 2 * rows * rank * (K + N))}
    requests = case["prompts"] + case["decode_rows"]
    adapters = _distinct(requests * served, case["pool"], case["alpha"])
    if case["alpha"] == 0.0 and case["prompts"] and case["prompts"] <= case["pool"]:
        adapters = case["prompts"] * served + _distinct(case["decode_rows"] * served, case["pool"], 0.0) * (1 - case["prompts"] / case["pool"])
    total, flops, seen = 0.0, 0.0, set()
    for name, shapes in _units(case):
        if name not in seen:
            seen.add(name)
            total += rows * shapes[0][0] * e
        for K, N in shapes:
            total += N * K * wb + rows * N * e + adapters * rank * (K + N) * ab
            flops += 2 * rows * K * N + served * rows * 2 * rank * (K + N)
    return {"bytes": case["layers"] * total, "flops": case["layers"] * flops}


def tolerance(case):
    # Four times what the path differs from the same sums in 64 bits: fp32 7e-7 and 5e-6 (K of 1000 to 1430); bf16, y
    # rounded once, 1.7e-3 and 5.4e-3, with a 4- or 8-bit base, whose weights are rounded to bf16, 2.3e-3 and 9.5e-3.
    return {"rel": 4e-6, "max": 2e-5} if case["dtype"] == "fp32" else {"rel": 8e-3, "max": 4e-2}
