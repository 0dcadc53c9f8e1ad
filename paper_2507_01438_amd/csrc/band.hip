// The matrix product of the GEMM path for a few hundred rows: y = x W^T + s B_i (A_i x) on tiles of 32 MA x 128 outputs, cut
// into K-slices until the launch fills the chip.
//
// The 256 x 256 tiles of gemm.hip leave most compute units idle here (one prompt of 389 rows x 4096 columns is 32 tiles)
// and multiply padding (389 rows -> 512).  So the height of a tile follows the batch, in steps of 32 rows up to 224; a
// tile is 128 columns wide; and K is cut into slices whose fp32 sums the last workgroup of a tile adds in slice order.
//   - x and W travel global -> LDS in whole cache lines through a ring of as many 64-wide K blocks as LDS holds (3 for
//     224 rows, up to 8): what bounds a launch of few rows is how many bytes of W are under way.
//   - 4 waves, 2 along the rows x 2 along the columns, 16 MA rows x 64 columns each with 16x16x32 matrix instructions
//     (the 32x32 form would need tiles in steps of 64 rows).  W is the first operand, so a lane holds four neighbouring
//     outputs of one row.
//   - a 4-bit or 8-bit W stays as it is in LDS; a fragment is converted on its way to the matrix cores.
//   - the expand B_i v_t comes after the K loop: every wave walks the runs of equal adapters in its own rows, all rows of a run
//     at a time where there are few, else 16 rows and 32 rank entries at a time through a ring of its own (no barriers), and a
//     row only takes what its own adapter gives.
//     Calls of up to 256 rows, which the decode kernel takes too, with fp32 shrink results, have these whole here as well:
//     three bf16 each (24 bits), three matrix instructions in the place of one, and the scale applied to what they give.
// A call with one adapter of rank 32 (route, shrink and product), on the 256 x 256 tiles / here: 389 rows 4096 x 4096 116 /
// 37 us, 4096 x 14336 121 / 72, 14336 x 4096 348 / 83; 1000 rows 4096 x 4096 121 / 57.  A K block of 224 x 128 takes 1330
// cycles (matrix instructions 900, LDS 1060); the first block lands after 7000, and from the last one to y it is 15500.
#include "gemm_common.h"

#include <algorithm>
#include <cmath>

using namespace elora;

namespace {

constexpr int BN = 128, BK = 64;
constexpr int kThreads = 256, kWaveCols = 64;
constexpr int kMaxMA = 7;
constexpr int kMaxSlices = 8;
constexpr int kRunsMost = 3;  // runs in a wave's rows, per K-slice, that are taken one after the other, over all of their rows
constexpr int kLdsBytes = 160 * 1024 - 512;  // (the rest: what the kernel declares by itself)

// everybody's loads up to N younger ones have landed, and everybody's LDS reads are over
template <int N> __device__ __forceinline__ void wait_and_meet() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory"); }

// LDS of a workgroup: `kDepth` stages of a K block each; after the K loop the same bytes are four rings, one per wave, of
// `kSteps` expand steps each.
template <int WFMT, int MA>
struct Band {
    static constexpr int kRows = MA * 32, kWaveRows = MA * 16;
    static constexpr int kXBytes = kRows * BK * 2;
    static constexpr int kWBytes = BN * BK * (WFMT == ELORA_W_SAME ? 4 : WFMT == ELORA_W_INT8_G32 ? 2 : 1) / 2;
    static constexpr int kScaleBytes = WFMT == ELORA_W_SAME ? 0 : BN * 4;  // a row's two fp16 scales
    static constexpr int kStage = kXBytes + kWBytes + kScaleBytes;
    static constexpr int kDepth = kLdsBytes / kStage < 8 ? kLdsBytes / kStage : 8;
    static constexpr int kWLoads = kWBytes / 4096;                         // per wave
    static constexpr int kLoads = MA + kWLoads + (kScaleBytes ? 1 : 0);    // per wave and K block
    // 16 rows of V, of its second and of its third parts, 64 columns of B_i, 32 rank entries
    static constexpr int kWholeLoads = 7, kRoundedLoads = 5, kStepBytes = kWholeLoads * 1024;
    // (all of LDS, unless the K loop leaves room for a second workgroup)
    static constexpr int kBytes = kDepth * kStage * 2 > kLdsBytes ? kLdsBytes / 4096 * 4096 : kDepth * kStage;
    // (four 16-byte zeros, 1024 apart, are read.  Less room for them would give tiles of 128 rows a fifth step; four / five:
    // gate + up of 256 rows of rank 16, 4096 x 14336, 168.4 / 170.6 us, of ranks 8 to 64 222 / 224, q + k + v of 500 180.4 / 179.7)
    static constexpr int kZeroBytes = 4096;
    static constexpr int kWaveBytes = (kBytes - kZeroBytes) / 4 / 1024 * 1024;
    static constexpr int kTableBytes = kWaveRows * (kMaxRank / 32) * 8;    // the wave's expand steps at most
    static constexpr int kStepRoom = (kWaveBytes - kTableBytes) / kStepBytes;
    static constexpr int kSteps = kStepRoom < 8 ? kStepRoom : 8;
    static_assert(kDepth >= 3 && kSteps >= 2 && kDepth * kLoads < 64 && kSteps * kWholeLoads < 64, "the load counter has six bits");
};

struct BandArgs {
    int T, K, N;
    int tiles_m, tiles_n, ks;
    const uint16_t *x;
    const void *W;
    const uint16_t *w_scales;
    const int32_t *row_slot;
    const float *row_scale;
    const uint16_t *V, *V_rest;  // V_rest: [2][T][Rpad] the second and third parts of the shrink results, or nullptr
    int Rpad;
    uint16_t *y;
    float *part;   // sums of K-slices: [tile][slice][wave][fragment][lane] x 4
    int *sync;
};

// kGather: for pools whose rows of B_i all have to be gathered (expand, below); takes any adapter, as the other does
template <int WFMT, int MA, bool kGather>
__global__ __launch_bounds__(kThreads) void lora_band_kernel(BandArgs ba, PoolView pool, int has_pool)
{
    typedef Band<WFMT, MA> G;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, m = lane & 15, g = lane >> 4;
    const int T = ba.T, K = ba.K, N = ba.N;
    if (blockIdx.x == 0 && tid == 0) ba.sync[kSyncShortRows] = 0;  // (what read it, the shrink, is over)
    // Workgroup b runs on XCD b % 8; an XCD takes a contiguous eighth of the list of (column tile, K-slice, row tile), so that
    // the row tiles that read the same piece of W run side by side and share it in the XCD's L2.
    const int units = ba.tiles_m * ba.tiles_n * ba.ks, per_xcd = (units + kXcds - 1) / kXcds;
    const int seq = (int)blockIdx.x / kXcds;
    int u = (int)blockIdx.x % kXcds * per_xcd + seq;
    if (seq >= per_xcd || u >= units) return;
    const int tm = u % ba.tiles_m;
    u /= ba.tiles_m;
    const int slice = u % ba.ks, tn = u / ba.ks, tile = tn * ba.tiles_m + tm;
    const int m0 = tm * G::kRows, n0 = tn * BN;
    const int r0 = m0 + wm * G::kWaveRows, c0 = n0 + wn * kWaveCols;  // the wave's corner of y

    // ---- K loop ------------------------------------------------------------------------------------------------------
    const unsigned blocks = (unsigned)K / BK;
    const int kb = (int)(blocks * (unsigned)slice / (unsigned)ba.ks);
    const int n_blk = (int)(blocks * (unsigned)(slice + 1) / (unsigned)ba.ks) - kb;
    // A direct load moves whole rows of a block: 8 rows of 128 bytes (x, bf16 W), 16 of 64 (8-bit W) or 32 of 32 (4-bit W).
    // A row's 16-byte chunks are permuted (chunk ^ row / 2, row / 4, row / 8) so that the fragment reads hit all banks.
    // Rows past the end of x and W repeat the last one; what they give is never stored.
    uint32_t xoff[MA], woff[G::kWLoads], soff = 0;
#pragma unroll
    for (int i = 0; i < MA; ++i) {
        const int row = 8 * (wave * MA + i) + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
        xoff[i] = (uint32_t)(((size_t)(min(m0 + row, T - 1) - m0) * K + chunk * 8) * 2);
    }
#pragma unroll
    for (int i = 0; i < G::kWLoads; ++i) {
        const int q = wave * G::kWLoads + i;
        if constexpr (WFMT == ELORA_W_SAME) {
            const int row = 8 * q + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
            woff[i] = (uint32_t)(((size_t)(min(n0 + row, N - 1) - n0) * K + chunk * 8) * 2);
        } else if constexpr (WFMT == ELORA_W_INT8_G32) {
            const int row = 16 * q + (lane >> 2), chunk = (lane & 3) ^ ((row >> 2) & 3);
            woff[i] = (uint32_t)((size_t)(min(n0 + row, N - 1) - n0) * K + chunk * 16);
        } else {
            const int row = 32 * q + (lane >> 1), chunk = (lane & 1) ^ ((row >> 3) & 1);
            woff[i] = (uint32_t)((size_t)(min(n0 + row, N - 1) - n0) * (K >> 1) + chunk * 16);
        }
    }
    if constexpr (WFMT != ELORA_W_SAME) soff = (uint32_t)((size_t)(min(n0 + (wave & 1) * 64 + lane, N - 1) - n0) * (K >> 5) * 2);
    const char *const xbase = reinterpret_cast<const char *>(ba.x + (size_t)m0 * K + (size_t)kb * BK);
    constexpr int kWRowBits = WFMT == ELORA_W_SAME ? 16 : WFMT == ELORA_W_INT8_G32 ? 8 : 4;
    const char *const wbase = static_cast<const char *>(ba.W) + ((size_t)n0 * K + (size_t)kb * BK) * kWRowBits / 8;
    const char *const sbase = reinterpret_cast<const char *>(ba.w_scales) + (((size_t)n0 * K + (size_t)kb * BK) >> 5) * 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
    // Column tiles and slices begin at different blocks: rows lie a multiple of the memory channels' pitch apart, and
    // workgroups that walk side by side would all ask the same channels (80 rows x 14336: 49.5 -> 45.7 us).
    const int turn = (int)((unsigned)(tn * ba.ks + slice) % (unsigned)n_blk);
    // load i of a block's kLoads
    auto issue_one = [&](int blk, int stage, auto ic_) __attribute__((always_inline)) {
        constexpr int i = decltype(ic_)::value;
        const uint32_t at = lds0 + (uint32_t)stage * G::kStage;
        blk += turn;
        if (blk >= n_blk) blk -= n_blk;
        if constexpr (i < MA) {
            dma16(at + (wave * MA + i) * 1024, xbase + (size_t)blk * (BK * 2), xoff[i]);
        } else if constexpr (i < MA + G::kWLoads) {
            dma16(at + G::kXBytes + (wave * G::kWLoads + i - MA) * 1024, wbase + (size_t)blk * (BK * kWRowBits / 8), woff[i - MA]);
        } else {
            // (waves 2 and 3 fetch the same scales once more: every wave has the same number of loads to count)
            dma4(at + G::kXBytes + G::kWBytes + (wave & 1) * 256, sbase + (size_t)blk * (BK / 32 * 2), soff);
        }
    };
    auto issue_block = [&](int blk, int stage) __attribute__((always_inline)) {
        static_for<0, G::kLoads>([&](auto i) __attribute__((always_inline)) { issue_one(blk, stage, i); });
    };

    floatx4 acc[MA][4];
#pragma unroll
    for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
            // (as values of their own: as copies of one zero the compiler finds no place for them in the loop, and moves every
            // sum between registers once per block: 389 rows x 4096 x 14336 112 us, without 87)
            asm volatile("" : "+a"(acc[a][b]));
        }

    // fragments of a 32-wide K step: rows of x, rows of W as they are stored; double-buffered
    typedef typename std::conditional<WFMT == ELORA_W_SAME, bf16x8, typename std::conditional<WFMT == ELORA_W_INT8_G32, u32x2, uint32_t>::type>::type wraw_t;
    bf16x8 xf[2][MA];
    wraw_t wf[2][4];
    uint16_t wsc[2][4];
    // fragment f of K step s of the block in `stage`: 0 .. 3 rows of W, 4 .. rows of x
    auto read_frag = [&](int to, int stage, int s, auto fc) __attribute__((always_inline)) {
        constexpr int f = decltype(fc)::value;
        const unsigned char *st = smem + stage * G::kStage;
        if constexpr (f >= 4) {
            xf[to][f - 4] = *reinterpret_cast<const bf16x8 *>(st + (wm * G::kWaveRows + (f - 4) * 16 + m) * 128 + (((s * 4 + g) ^ ((m >> 1) & 7)) * 16));
        } else {
            const int row = wn * kWaveCols + f * 16 + m;
            const unsigned char *w = st + G::kXBytes;
            if constexpr (WFMT == ELORA_W_SAME) {
                wf[to][f] = *reinterpret_cast<const wraw_t *>(w + row * 128 + (((s * 4 + g) ^ ((m >> 1) & 7)) * 16));
            } else {
                if constexpr (WFMT == ELORA_W_INT8_G32) wf[to][f] = *reinterpret_cast<const wraw_t *>(w + row * 64 + (((s * 2 + (g >> 1)) ^ ((m >> 2) & 3)) * 16) + (g & 1) * 8);
                else wf[to][f] = *reinterpret_cast<const wraw_t *>(w + row * 32 + ((s ^ ((m >> 3) & 1)) * 16) + g * 4);
                wsc[to][f] = *reinterpret_cast<const uint16_t *>(w + G::kWBytes + row * 4 + s * 2);
            }
        }
    };
    auto w_operand = [&](int from, int b) __attribute__((always_inline)) {
        if constexpr (WFMT == ELORA_W_SAME) return wf[from][b];
        else if constexpr (WFMT == ELORA_W_INT8_G32) return __builtin_bit_cast(bf16x8, q8_to_bf16x8(wf[from][b], fp16_to_f32(wsc[from][b])));
        else return __builtin_bit_cast(bf16x8, w4_to_bf16x8(wf[from][b], fp16_to_f32(wsc[from][b])));
    };
    // One K step: 4 MA matrix instructions on the fragments `from`.  Behind those of the first half the fragments of the
    // next step are read, behind those of the second half the next block's direct loads are issued, a few per slot: a
    // matrix instruction keeps its pipe busy for 16 cycles, during which the wave issues what else it has to.
    constexpr int kFirstLoads = (G::kLoads + 1) / 2;
    auto k_step = [&](auto from_c, int rstage, int rs, int lblk, int lstage) __attribute__((always_inline)) {
        constexpr int from = decltype(from_c)::value;
        constexpr int kSlots = 4 * MA, kHalf = kSlots / 2, kReads = MA + 4;
        // (the first half of a block's loads in step 1, the second half in step 0 of the next block)
        constexpr int kFirst = from == 1 ? 0 : kFirstLoads, kLoads = from == 1 ? kFirstLoads : G::kLoads - kFirstLoads;
        bf16x8 w = w_operand(from, 0);
        static_for<0, kSlots>([&](auto ec) __attribute__((always_inline)) {
            constexpr int e = decltype(ec)::value, b = e / MA, a = e % MA;
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, xf[from][a], acc[a][b], 0, 0, 0);
            if constexpr (a == MA - 1 && b < 3) w = w_operand(from, b + 1);
            if constexpr (e < kHalf) static_for<e * kReads / kHalf, (e + 1) * kReads / kHalf>([&](auto f) __attribute__((always_inline)) { read_frag(from ^ 1, rstage, rs, f); });
            else static_for<(e - kHalf) * kLoads / kHalf, (e + 1 - kHalf) * kLoads / kHalf>([&](auto i) __attribute__((always_inline)) { issue_one(lblk, lstage, ic<kFirst + decltype(i)::value>{}); });
            if constexpr (WFMT == ELORA_W_SAME) __builtin_amdgcn_sched_barrier(0);
        });
        // (a W that is converted on the way: a few vector instructions behind every matrix instruction, not all in a row)
        if constexpr (WFMT != ELORA_W_SAME)
            static_for<0, kSlots>([&](auto) __attribute__((always_inline)) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            });
        __builtin_amdgcn_sched_barrier(0);
    };

    // the slots, scales and ranks of the wave's rows (the ranks are on their way during the K loop)
    const bool whole = ba.V_rest != nullptr;
    int slot_v[2] = {INT32_MIN, INT32_MIN}, rank_v[2] = {0, 0};
    float scale_v[2] = {1.0f, 1.0f};  // (V that is rounded has the scale in it)
    if (has_pool) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (h * 64 + lane < G::kWaveRows && r0 + h * 64 + lane < T) {
                slot_v[h] = ba.row_slot[r0 + h * 64 + lane];
                if (whole) scale_v[h] = ba.row_scale[r0 + h * 64 + lane];
            }
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (slot_v[h] >= 0) rank_v[h] = pool.meta[slot_v[h]].rank;
    }
#pragma unroll 1
    for (int i = 0; i < G::kDepth - 1; ++i) issue_block(min(i, n_blk - 1), i);
    // (the loop's first turn asks for the second half of block kDepth - 1)
    static_for<0, kFirstLoads>([&](auto i) __attribute__((always_inline)) { issue_one(min(G::kDepth - 1, n_blk - 1), G::kDepth - 1, i); });
    wait_and_meet<(G::kDepth - 2) * G::kLoads + kFirstLoads>();
    static_for<0, MA + 4>([&](auto f) __attribute__((always_inline)) { read_frag(0, 0, 0, f); });
    // One loop, in which nothing depends on how much is left: the last blocks ask for the last block once more, into stages
    // that nobody reads again.
    int stage = 0, before = G::kDepth - 1;  // (the stage of the block before, which block blk + kDepth - 1 goes into)
    for (int blk = 0; blk < n_blk; ++blk) {
        const int next = stage + 1 == G::kDepth ? 0 : stage + 1;
        k_step(ic<0>{}, stage, 1, min(blk + G::kDepth - 1, n_blk - 1), before);
        wait_and_meet<(G::kDepth - 2) * G::kLoads>();  // block blk + 1 has landed, and the stage of block blk has been read
        k_step(ic<1>{}, next, 0, min(blk + G::kDepth, n_blk - 1), stage);
        before = stage;
        stage = next;
    }
    wait_loads<0>();

    // ---- expand ------------------------------------------------------------------------------------------------------------
    // Few runs of equal adapters in the wave's rows (prompts; up to kRunsMost): a run and 32 rank entries at a time, over all of
    // its 16-row blocks: 4 KiB of B_i and 1 KiB of V per block straight into registers, all at once, the next ones on their way
    // meanwhile.  (389 rows of one adapter, 4096 x 14336, from the end of the K loop to y: 23000 cycles in steps of one block,
    // which each waited for loads of the same B_i and for the stores of the block before, so 15000.  A tile's K-slices take turns at the
    // runs.)
    // Otherwise a step is (16-row block, run of equal adapters in it, 32 rank entries): 1 or 3 KiB of V and 4 of B_i for four or
    // twelve matrix instructions; a tile's K-slices take turns at the runs.  The wave first writes its steps out as a table, a lane per row;
    // the loads of kSteps - 1 steps are under way while one is multiplied.  Ranks that are no multiples of 8, and adapters in
    // 8-bit blocks, have rows of B_i that a 16-byte load cannot take: their fragments are gathered when the step is due, in a
    // loop of their own.  What bounds the plain steps is instructions and waits, with one wave per SIMD: 120 instructions a step
    // (the gathered ones 230), and no stores of y between them, whose acknowledgements the loads behind them would wait for
    // (150 rows of mixed rank, 4096 x 14336: 75 -> 66 us).
    // The code is kept short: the blocks go through one loop, always as acc[0], and the others move up behind each.  (A
    // switch over the blocks made the compiler copy all sums at every step: 2050 cycles a step; unrolled, 389 rows of one
    // adapter took 3000.)
    int n_steps = 0, first[2] = {0, 0};  // (first: steps before the lane's row)
    unsigned char *const own = smem + wave * G::kWaveBytes;
    uint64_t *const table = reinterpret_cast<uint64_t *>(own + G::kSteps * G::kStepBytes);
    struct Step {
        int row, end, j0, rank, slot;
    };
    auto step_at = [&](int i) __attribute__((always_inline)) {
        const u32x2 r = *reinterpret_cast<const u32x2 *>(table + min(i, n_steps - 1));
        const int a = __builtin_amdgcn_readfirstlane(r[0]), slot = __builtin_amdgcn_readfirstlane(r[1]);
        return Step{a & 255, (a >> 8) & 255, ((a >> 16) & 15) * 32, a >> 20, slot};
    };
    const bool q8 = pool.q8 != 0;
    const uint32_t ring0 = lds0 + (uint32_t)(wave * G::kWaveBytes);
    const char *const vbase = reinterpret_cast<const char *>(ba.V + (size_t)r0 * ba.Rpad), *const vmid = reinterpret_cast<const char *>(ba.V_rest + (size_t)r0 * ba.Rpad),
               *const vlast = vmid + (size_t)T * ba.Rpad * 2;
    const int line = lane >> 2, chunk = (lane & 3) ^ ((line >> 2) & 3);
    uint32_t col[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) col[i] = (uint32_t)min(c0 + i * 16 + line, N - 1);
    auto issue = [&](const Step &st, int at) __attribute__((always_inline)) {
        const uint32_t lds = ring0 + (uint32_t)at * G::kStepBytes;
        const int row = min((st.row & ~15) + line, T - 1 - r0);
        const uint32_t voff = (uint32_t)((row * ba.Rpad + st.j0 + chunk * 8) * 2);
        dma16(lds, vbase, voff);
        if (whole) {
            dma16(lds + 1024, vmid, voff);
            dma16(lds + 2048, vlast, voff);
        }
        // (a gathered step loads its row of V again, so that all steps have the same number of loads)
        const bool gather = q8 || (st.rank & 7) != 0;
        const char *const Bm = gather ? vbase : slot_B(pool, st.slot);
        const uint32_t j = gather ? voff : 2u * (uint32_t)(st.j0 + chunk * 8 < st.rank ? st.j0 + chunk * 8 : st.j0);
        const uint32_t stride = gather ? 0u : 2u * (uint32_t)st.rank;
#pragma unroll
        for (int i = 0; i < 4; ++i) dma16(lds + 3072 + i * 1024, Bm, col[i] * stride + j);
    };
    // The same loads for a wave whose steps are all plain ones (ranks that are multiples of 8, no 8-bit blocks): its table holds
    // the adapter's place in the pool instead of the slot, in units of 256 bytes.
    const char *const slots0 = pool.slots;
    auto issue_plain = [&](int w0, int w1, int at, auto whole_c) __attribute__((always_inline)) {
        const uint32_t lds = ring0 + (uint32_t)at * G::kStepBytes;
        const uint32_t j0 = (uint32_t)((w0 >> 16) & 15) * 32, rank = (uint32_t)(w0 >> 20);
        const int row = min((w0 & 0xf0) + line, T - 1 - r0);
        const uint32_t voff = __umul24(row, 2u * ba.Rpad) + (2u * j0 + 16u * chunk);
        dma16(lds, vbase, voff);
        if constexpr (decltype(whole_c)::value) {
            dma16(lds + 1024, vmid, voff);
            dma16(lds + 2048, vlast, voff);
        }
        const char *const Bm = slots0 + ((uint64_t)(uint32_t)w1 << 8);
        const uint32_t j = j0 + 8u * chunk, jb = 2u * (j < rank ? j : j0);
#pragma unroll
        for (int i = 0; i < 4; ++i) dma16(lds + 3072 + i * 1024, Bm, __umul24(col[i], 2u * rank) + jb);
    };
    bool plain = false, in_runs = false;
    if (has_pool) {
        const int before0 = __shfl_up(slot_v[0], 1), before1 = __shfl_up(slot_v[1], 1), last0 = __builtin_amdgcn_readlane(slot_v[0], 63);
        const bool cut = (lane & 15) == 0;
        const uint64_t starts[2] = {__ballot(cut || slot_v[0] != before0), __ballot(cut || slot_v[1] != (lane == 0 ? last0 : before1))};
        const uint64_t run[2] = {starts[0] & __ballot(rank_v[0] > 0), starts[1] & __ballot(rank_v[1] > 0)};  // first rows of runs with an adapter
        if constexpr (!kGather) {
            plain = !q8 && (__ballot(((rank_v[0] | rank_v[1]) & 7) != 0)) == 0;
            // ---- few runs in the wave's rows (prompts): a run and 32 rank entries at a time, over all of its 16-row blocks
            uint64_t left[2] = {__ballot(lane == 0 || slot_v[0] != before0) & run[0], __ballot(slot_v[1] != (lane == 0 ? last0 : before1)) & run[1]};
            in_runs = plain && !whole && (int)__popcll(left[0]) + (int)__popcll(left[1]) <= kRunsMost * ba.ks;
            if (in_runs) {
                const uint64_t ends[2] = {__ballot(slot_v[0] != before0), __ballot(slot_v[1] != (lane == 0 ? last0 : before1))};  // (lane 0 of the first: no matter)
                int lo = 0, hi = 0, rank = 0, j0 = 0;  // the run and the entries whose fragments come next
                int others = slice;                    // runs that fall to other slices before the next one of this slice
                const uint16_t *Bm = nullptr;
                auto next = [&]() __attribute__((always_inline)) {
                    j0 += 32;
                    if (j0 < rank) return true;
                    for (; others > 0 && (left[0] | left[1]) != 0; --others) left[left[0] == 0] &= left[left[0] == 0] - 1;
                    if ((left[0] | left[1]) == 0) return false;
                    others = ba.ks - 1;
                    const int h = left[0] == 0, l = (int)__builtin_ctzll(left[h]);
                    left[h] &= left[h] - 1;
                    lo = h * 64 + l;
                    const uint64_t after0 = h == 0 && l < 63 ? ends[0] & (~0ull << (l + 1)) : 0, after1 = h == 0 ? ends[1] : l < 63 ? ends[1] & (~0ull << (l + 1)) : 0;
                    hi = after0 ? (int)__builtin_ctzll(after0) : after1 ? 64 + (int)__builtin_ctzll(after1) : 128;
                    rank = h == 0 ? __builtin_amdgcn_readlane(rank_v[0], l) : __builtin_amdgcn_readlane(rank_v[1], l);
                    Bm = reinterpret_cast<const uint16_t *>(slot_B(pool, h == 0 ? __builtin_amdgcn_readlane(slot_v[0], l) : __builtin_amdgcn_readlane(slot_v[1], l)));
                    j0 = 0;
                    return true;
                };
                u32x4 vf[MA], bf[4];
                auto load = [&]() __attribute__((always_inline)) {
                    const int j = j0 + g * 8;
#pragma unroll
                    for (int b = 0; b < 4; ++b) bf[b] = *reinterpret_cast<const u32x4 *>(Bm + (uint32_t)min(c0 + b * 16 + m, N - 1) * (uint32_t)rank + (uint32_t)(j < rank ? j : j0));
#pragma unroll
                    for (int a = 0; a < MA; ++a) vf[a] = *reinterpret_cast<const u32x4 *>(ba.V + (size_t)min(r0 + a * 16 + m, T - 1) * ba.Rpad + j);
                };
                bool more = next();
                if (more) load();
#pragma unroll 1
                while (more) {
                    const int lo_ = lo, hi_ = hi;
                    const bool cut_off = j0 + g * 8 >= rank;
                    bf16x8 v[MA], bm[4];
#pragma unroll
                    for (int b = 0; b < 4; ++b) bm[b] = __builtin_bit_cast(bf16x8, cut_off ? u32x4{0, 0, 0, 0} : bf[b]);
#pragma unroll
                    for (int a = 0; a < MA; ++a) v[a] = __builtin_bit_cast(bf16x8, vf[a]);
                    more = next();
                    if (more) load();
#pragma unroll
                    for (int a = 0; a < MA; ++a) {
                        if (a * 16 >= hi_ || a * 16 + 16 <= lo_) continue;
                        if (lo_ <= a * 16 && hi_ >= min(a * 16 + 16, T - r0)) {
#pragma unroll
                            for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[b], v[a], acc[a][b], 0, 0, 0);
                        } else {
                            const bool in = (a * 16 + m >= lo_) & (a * 16 + m < hi_);  // (a row of another run takes nothing, not even zero times this adapter)
#pragma unroll
                            for (int b = 0; b < 4; ++b) {
                                const floatx4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[b], v[a], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                                for (int q = 0; q < 4; ++q) acc[a][b][q] += in ? d[q] : 0.0f;
                            }
                        }
                    }
                }
            }
        }
        __syncthreads();  // every wave is done with the stages
        if (!kGather && tid < 16) *reinterpret_cast<uint32_t *>(smem + 4 * G::kWaveBytes + (tid >> 2) * 1024 + (tid & 3) * 4) = 0;  // (read by every wave: the barrier below)
#pragma unroll
        for (int h = 0; h < (G::kWaveRows + 63) / 64; ++h) {
            const uint64_t below = (1ull << lane) - 1;
            const int number = (int)__popcll(run[h] & below) + (h ? (int)__popcll(run[0]) : 0);
            const int n = ((run[h] >> lane) & 1) && !in_runs && number % ba.ks == slice ? (rank_v[h] + 31) >> 5 : 0;
            int upto = n;  // steps of the rows up to this one
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int v = __shfl_up(upto, d);
                if (lane >= d) upto += v;
            }
            first[h] = n_steps + upto - n;
            const uint64_t after = lane == 63 ? 0 : starts[h] & (~0ull << (lane + 1));
            const int row = h * 64 + lane, end = h * 64 + (after ? (int)__builtin_ctzll(after) : 64);
            // step record: first row | end row << 8 | 32 entries number << 16 | rank << 20, slot
            for (int i = 0; i < n; ++i)
                table[first[h] + i] = (uint64_t)(uint32_t)(row | (end << 8) | (i << 16) | (rank_v[h] << 20)) |
                                      ((uint64_t)(plain ? (uint32_t)((slot_v[h] * pool.slot_bytes + pool.b_offset) >> 8) : (uint32_t)slot_v[h]) << 32);
            n_steps += __builtin_amdgcn_readlane(upto, 63);
        }
        if constexpr (kGather) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (a wave reads what its own lanes wrote)
        else __syncthreads();
        if (n_steps > 0) {
#pragma unroll 1
            for (int i = 0; i < G::kSteps - 1; ++i) {
                if (!plain) {
                    issue(step_at(i), i);
                } else {
                    const u32x2 r = *reinterpret_cast<const u32x2 *>(table + min(i, n_steps - 1));
                    const int w0 = __builtin_amdgcn_readfirstlane(r[0]), w1 = __builtin_amdgcn_readfirstlane(r[1]);
                    if (whole) issue_plain(w0, w1, i, std::true_type{});
                    else issue_plain(w0, w1, i, std::false_type{});
                }
            }
        }
    }
    // sums of K-slices, written through to memory and read past the first-level cache (nothing depends on where a tile's
    // workgroups run)
    constexpr int kFrags = MA * 4, kCoherent = 16;  // sc1
    auto rsrc = __builtin_amdgcn_make_buffer_rsrc(ba.part + (size_t)tile * ba.ks * (4 * kFrags * 256), 0, ba.ks * (4 * kFrags * 1024), 0x00020000);
    const int part_at = wave * kFrags * 1024 + lane * 16, slice_bytes = 4 * kFrags * 1024;
    // block a of y, or of the slice's sums, from acc[at]: a lane has four neighbouring outputs of row m
    auto store_block = [&](int a, int at) __attribute__((always_inline)) {
        const int row = r0 + a * 16 + m;
        uint16_t *const yrow = ba.y + (size_t)row * N;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int c = c0 + b * 16 + g * 4;
            if (row < T && c < N) *reinterpret_cast<u32x2 *>(yrow + c) = u32x2{pack_bf16x2(acc[at][b][0], acc[at][b][1]), pack_bf16x2(acc[at][b][2], acc[at][b][3])};
        }
    };
    auto store_part = [&](int a, int at) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[at][b]), rsrc, part_at + a * 4096 + b * 1024, slice * slice_bytes, kCoherent);
    };
    auto store_y = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < MA; ++a) store_block(a, a);
    };
    int step = 0, at = 0;
    // What a step of a plain wave costs is instructions and the waits between them (one wave per SIMD): the table entries are
    // read a step ahead, the rows' sums stay in vector registers, and a row outside the run is masked off as a lane.
    u32x2 rec_now{0, 0}, rec_next{0, 0};  // this step's entry; that of the step to ask for
    auto fetch_records = [&](int step) __attribute__((always_inline)) {
        rec_now = *reinterpret_cast<const u32x2 *>(table + min(step, n_steps - 1));
        rec_next = *reinterpret_cast<const u32x2 *>(table + min(step + G::kSteps - 1, n_steps - 1));
    };
    if (plain && n_steps > 0) fetch_records(0);
    const uint32_t zero_at = (uint32_t)(4 * G::kWaveBytes);
    auto plain_steps = [&](int a, int stop, float row_scale, auto whole_c) __attribute__((always_inline)) {
        constexpr bool kWhole = decltype(whole_c)::value;
        floatx4 sum[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            sum[b] = acc[0][b];
            asm volatile("" : "+v"(sum[b]));
        }
        const int row = a * 16 + m;
#pragma unroll 1
        for (; step < stop; ++step) {
            const int w0 = __builtin_amdgcn_readfirstlane(rec_now[0]);
            const int n0_ = __builtin_amdgcn_readfirstlane(rec_next[0]), n1_ = __builtin_amdgcn_readfirstlane(rec_next[1]);
            issue_plain(n0_, n1_, at == 0 ? G::kSteps - 1 : at - 1, whole_c);
            fetch_records(step + 1);
            wait_loads<(kWhole ? G::kWholeLoads : G::kRoundedLoads) * (G::kSteps - 1)>();
            const uint32_t st = (uint32_t)(wave * G::kWaveBytes) + (uint32_t)at * G::kStepBytes + (uint32_t)(m * 64 + (g ^ ((m >> 2) & 3)) * 16);
            const int rank = w0 >> 20, j = ((w0 >> 16) & 15) * 32 + g * 8;
            // (entries past the rank: zero in V; zero here too, whatever the adapter holds)
            const unsigned char *const bp = smem + (j < rank ? st + 3072 : zero_at);
            bf16x8 v[kWhole ? 3 : 1], bm[4];
#pragma unroll
            for (int q = 0; q < (kWhole ? 3 : 1); ++q) v[q] = *reinterpret_cast<const bf16x8 *>(smem + st + q * 1024);
#pragma unroll
            for (int b = 0; b < 4; ++b) bm[b] = *reinterpret_cast<const bf16x8 *>(bp + b * 1024);
            floatx4 d[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) d[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[b], v[0], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            if constexpr (kWhole) {
#pragma unroll
                for (int b = 0; b < 4; ++b) d[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[b], v[1], d[b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < 4; ++b) d[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[b], v[2], d[b], 0, 0, 0);
            }
            if ((row >= (w0 & 255)) & (row < ((w0 >> 8) & 255))) {  // (a row of another run takes nothing, not even zero times this adapter)
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q) sum[b][q] = kWhole ? fmaf(d[b][q], row_scale, sum[b][q]) : sum[b][q] + d[b][q];
            }
#pragma unroll
            for (int b = 0; b < 4; ++b) asm volatile("" : "+v"(sum[b]));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (this step's place has been read)
            at = at + 1 == G::kSteps ? 0 : at + 1;
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[0][b] = sum[b];
    };
    if (n_steps > 0) {
#pragma unroll 1
    for (int a = 0; a < MA; ++a) {
        float row_scale = 1.0f;
        if (whole) row_scale = __shfl(a < 4 ? scale_v[0] : scale_v[1], (a & 3) * 16 + m);
        const int stop = a + 1 == MA ? n_steps : __builtin_amdgcn_readlane(a + 1 < 4 ? first[0] : first[1], ((a + 1) & 3) * 16);
        if (plain) {
            if (whole) plain_steps(a, stop, row_scale, std::true_type{});
            else plain_steps(a, stop, row_scale, std::false_type{});
        }
#pragma unroll 1
        for (; step < stop; ++step) {
            const Step cur = step_at(step);
            // (the place read a step ago; behind the last step its loads are asked for again, so that the count stays)
            issue(step_at(step + G::kSteps - 1), at == 0 ? G::kSteps - 1 : at - 1);
            if (whole) wait_loads<G::kWholeLoads *(G::kSteps - 1)>();
            else wait_loads<G::kRoundedLoads *(G::kSteps - 1)>();
            const unsigned char *const st = own + at * G::kStepBytes;
            const int place = (g ^ ((m >> 2) & 3)) * 16, j = cur.j0 + g * 8;
            bf16x8 v = *reinterpret_cast<const bf16x8 *>(st + m * 64 + place), bm[4];
            const u32x4 zero{0, 0, 0, 0};
#pragma unroll
            for (int b = 0; b < 4; ++b) bm[b] = *reinterpret_cast<const bf16x8 *>(st + 3072 + (b * 16 + m) * 64 + place);
            if (q8 || (cur.rank & 7) != 0) {
                const char *const Bm = slot_B(pool, cur.slot);
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const size_t e = (size_t)min(c0 + b * 16 + m, N - 1) * cur.rank + j;
                    u32x4 o = zero;
                    if (q8) {
                        if (j < cur.rank) o = q8_to_bf16x8(*reinterpret_cast<const u32x2 *>(Bm + e), fp16_to_f32(slot_B_scales(pool, cur.slot)[e >> 5]));
                    } else {
                        const uint16_t *const src = reinterpret_cast<const uint16_t *>(Bm) + e;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const uint32_t lo = j + 2 * q < cur.rank ? src[2 * q] : 0u, hi = j + 2 * q + 1 < cur.rank ? src[2 * q + 1] : 0u;
                            o[q] = lo | (hi << 16);
                        }
                    }
                    // (waited for here: behind the branch, the wait would be one of every step, and for all loads under way)
                    asm volatile("" : "+v"(o));
                    bm[b] = __builtin_bit_cast(bf16x8, o);
                }
            }
            if (j >= cur.rank) {  // (entries past the rank: zero in V; zero here too, whatever the adapter holds)
                v = __builtin_bit_cast(bf16x8, zero);
#pragma unroll
                for (int b = 0; b < 4; ++b) bm[b] = __builtin_bit_cast(bf16x8, zero);
            }
            const int row = a * 16 + m;
            const bool in = row >= cur.row && row < cur.end;  // (a row of another run takes nothing, not even zero times this adapter)
            floatx4 d[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) d[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[b], v, floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            if (whole) {
                const bf16x8 mid = *reinterpret_cast<const bf16x8 *>(st + 1024 + m * 64 + place), last = *reinterpret_cast<const bf16x8 *>(st + 2048 + m * 64 + place);
#pragma unroll
                for (int b = 0; b < 4; ++b) d[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[b], mid, d[b], 0, 0, 0);
#pragma unroll
                for (int b = 0; b < 4; ++b) d[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm[b], last, d[b], 0, 0, 0);
            }
            const float scale = in ? row_scale : 0.0f;
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[0][b][q] = fmaf(in ? d[b][q] : 0.0f, scale, acc[0][b][q]);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (this step's place has been read)
            at = at + 1 == G::kSteps ? 0 : at + 1;
        }
        if constexpr (kGather) {
            if (ba.ks == 1) store_block(a, 0);
            else store_part(a, 0);
        }
        // (the blocks move up, round the circle: as many turns as there are blocks put every one back)
        floatx4 top[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) top[b] = acc[0][b];
#pragma unroll
        for (int i = 0; i + 1 < MA; ++i)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[i][b] = acc[i + 1][b];
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[MA - 1][b] = top[b];
    }
    }
    wait_loads<0>();  // (also those asked for behind the last step: they land before the LDS is given back)
    const bool stored = kGather && n_steps > 0;
    if (ba.ks == 1) {
        if (!stored) store_y();
        return;
    }
    if (!stored) {
#pragma unroll
        for (int a = 0; a < MA; ++a) store_part(a, a);
    }

    // ---- sums of the K-slices: the last workgroup of the tile to come adds them, in slice order -----------------------------
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's sums have reached memory
    __syncthreads();
    if (tid == 0) {
        const int before_me = __hip_atomic_fetch_add(&ba.sync[kSyncTiles + tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = before_me == ba.ks - 1;
        if (s_last) __hip_atomic_store(&ba.sync[kSyncTiles + tile], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!s_last) return;
    // (its own sums as well: the order of the additions does not depend on who comes last)
#pragma unroll
    for (int f = 0; f < kFrags; ++f) acc[f >> 2][f & 3] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int k = 0; k < ba.ks; ++k) {
        u32x4 w[kFrags];
#pragma unroll
        for (int f = 0; f < kFrags; ++f) w[f] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, part_at + f * 1024, k * slice_bytes, kCoherent);
#pragma unroll
        for (int f = 0; f < kFrags; ++f) acc[f >> 2][f & 3] += __builtin_bit_cast(floatx4, w[f]);
    }
    store_y();
}

int g_mode = -1, g_mode_tiles = 0, g_mode_slices = 0;  // (elora_debug_band)

}  // namespace

void elora::band_set(int mode, int tiles_m, int slices)
{
    g_mode = mode;
    g_mode_tiles = tiles_m;
    g_mode_slices = slices;
}

// Which tiles, and whether this kernel or the 256 x 256 tiles: the launch's time in cycles, from what a K block, a tile's
// beginning and end, a step of the expand and the sums of slices were measured to take, times the rounds of 256 workgroups
// (one per compute unit).
//   here: a K block 270 + 160 ma (a W that is converted on the way 1550 + 105 ma), a tile 6000 + 2300 ma, an expand step
//   1600 (adapters in 8-bit blocks 6500), the slices' sums 2000 + 450 ma each; 20 % more than that where there is more than
//   one round;
//   (the step of 1600 is from when it took 230 instructions, not the 120 that plain adapters take now: with an adapter per row
//   this kernel stays the faster one beyond where the rule ends, there / here: 1000 rows of rank 64, 2560 x 7680, 513 / 284 us,
//   3000 rows 4096 x 4096 661 / 454, 2000 of rank 16, 1024 x 1024, 98 / 82)
//   there: a K block 3300, in further rounds 2900 (from the bf16 copy of W 2600, converted on the way 5700), a tile 6000, 16
//   rank entries of a short run 850 (adapters in 8-bit blocks 4000), the copy 1.04e-3 per weight.
// Over 1488 calls of 300 to 4000 rows (eight W of 512 x 512 to 14336 x 4096 and 4096 x 14336, one prompt to a row per adapter,
// ranks 8 to 128, all storage formats) the choice is slower than the 256 x 256 tiles by more than 3 % in 4 and by 9 % at most;
// the mean call takes 68 % of its time there (measured with the constants).  (Asking for the estimate to be 8 % lower is what keeps these from being 27.)
// (4096 x 14336, here / there: 600 rows of one adapter 109 / 119 us, 800 of two 124 / 119, 1800 235 / 208, 600 of an adapter
// each 217 / 188; 4096 x 4096: 600 of an adapter each 103 / 185, 1000 of one 58 / 121; 2560 x 7680, 3000 rows: 171 / 140.)
bool elora::band_shape(const BandCall &c, size_t part_bytes, BandShape *s)
{
    const int T = c.T, K = c.K, N = c.N;
    if (g_mode == 0 || K % BK != 0 || N % 8 != 0) return false;
    const int tiles_n = (N + BN - 1) / BN, blocks = K / BK;
    const int least = (T + 32 * kMaxMA - 1) / (32 * kMaxMA);
    auto rounds = [](double workgroups) { return std::ceil(workgroups / 256); };
    // the cheapest tiles of this kernel, on W as it is stored or on a bf16 copy of it (the copy itself not counted); negative: none
    auto cheapest = [&](bool from_copy, BandShape *to) {
        double best = -1.0;
        for (int tiles_m = g_mode_tiles > least ? g_mode_tiles : least; tiles_m <= (g_mode_tiles ? g_mode_tiles : least + 2); ++tiles_m) {
            const int ma = ((T + tiles_m - 1) / tiles_m + 31) / 32, tm = (T + 32 * ma - 1) / (32 * ma);
            const double block = c.wfmt == ELORA_W_SAME || from_copy ? 270 + 160 * ma : 1550 + 105 * ma;
            // a wave's steps: where the runs are spread over the batch, and what the tile with most of them has above that
            const double row = (c.q8 ? 6500.0 : 1600.0) * c.pieces32;
            const double spread = row * 16 * ma * c.runs / T, above = std::max(0.0, row * std::min(16 * ma, c.runs) - spread);
            for (int ks = g_mode_slices ? g_mode_slices : 1; ks <= (g_mode_slices ? g_mode_slices : kMaxSlices); ++ks) {
                if (ks > blocks || (ks > 1 && ((long long)tm * tiles_n > kSyncTileCount || (size_t)tm * tiles_n * ks * (ma * 32 * BN * 4) > part_bytes))) continue;
                const double n = rounds((double)tm * tiles_n * ks);
                const double tile = (blocks + ks - 1) / ks * block + 6000 + 2300 * ma + spread / ks;
                const double cycles = (n * tile + above / ks) * (n > 1 ? 1.2 : 1.0) + (ks > 1 ? 2000 + 450.0 * ks * ma : 0);
                if (best < 0 || cycles < best) {
                    best = cycles;
                    *to = BandShape{ma, tm, ks, from_copy};
                }
            }
        }
        return best;
    };
    double best = cheapest(false, s), copy = c.copied ? 1.04e-3 * K * N : 0.0;
    if (best < 0 || g_mode == 1 || c.only) return best >= 0;
    // On the copy that the 256 x 256 tiles would run on, where there is room for one: next to it a converted W costs about 18000
    // cycles a launch more than its blocks do.  A copy that does not stay in the caches costs more to make and to read, and
    // has to be the better one by a sixth.  (One or two prompts, 8-bit W, as stored / on the copy: 389 rows 4096 x 4096 57 / 45 us,
    // 14336 x 4096 110 / 122 (stored), 1000 rows 4096 x 4096 86 / 59, 14336 x 4096 243 / 170, 2000 rows 6144 x 2048 123 / 79, 2048 x 2048
    // 61 / 42; 300 rows 4096 x 4096 48 / 41, where a group's second copy, a launch of its own, takes that back.)
    const double weights = (double)K * N, in_cache = 32e6;
    if (c.copied && T >= 320) {
        BandShape from_copy;
        const double made = 1.04e-3 * weights + 0.6e-3 * std::max(0.0, weights - in_cache), on_copy = cheapest(true, &from_copy) + made;
        if (on_copy < (weights > in_cache ? 0.83 : 1.0) * (best + 18000)) {
            best = on_copy;
            copy = made;
            *s = from_copy;
        }
    }
    // (The 18000 stay out of what follows: they would send 30 of 40000 drawn calls to the 256 x 256 tiles, of which twelve were
    // timed.  Ten are faster here, 413 rows of 50 prompts 6144 x 11008 8-bit 161 / 170 us, 376 of 8 2560 x 14336 83 / 96, and two
    // slower by 2 and 3 %.)
    const double n = rounds((double)((T + 255) / 256) * ((N + 255) / 256));
    const double block = c.copied ? 2600 : c.wfmt != ELORA_W_SAME ? 5700 : n > 1 ? 2900 : 3300;
    // (the most that a wave of a tile has, 128 rows; where the runs are spread over the batch, every round's tiles have them)
    const double run = (c.q8 ? 4000.0 : 850.0) * c.pieces16, spread = c.runs < T ? run * 128 * c.runs / T : run * 128, above = std::max(0.0, run * std::min(128, c.runs) - spread);
    return best < 0.92 * (n * (blocks * block + 6000 + spread) + above + copy);
}

bool elora::band_whole(const LinearArgs &a) { return a.has_pool && a.T <= kWholeRows && a.wsl.v_rest_bytes != 0; }

int elora::enqueue_band(const LinearArgs &a, const BandShape &s, hipStream_t stream)
{
    BandArgs b;
    b.T = a.T;
    b.K = a.K;
    b.N = a.N;
    b.tiles_m = s.tiles_m;
    b.tiles_n = (a.N + BN - 1) / BN;
    b.ks = s.ks;
    b.x = static_cast<const uint16_t *>(a.x);
    b.W = s.copied ? static_cast<const void *>(a.ws + a.wsl.wdeq) : a.W;
    b.w_scales = static_cast<const uint16_t *>(a.w_scales);
    b.row_slot = reinterpret_cast<const int32_t *>(a.ws + a.wsl.row_slot);
    b.V = reinterpret_cast<const uint16_t *>(a.ws + a.wsl.v);
    b.V_rest = band_whole(a) ? reinterpret_cast<const uint16_t *>(a.ws + a.wsl.v_rest) : nullptr;
    b.row_scale = reinterpret_cast<const float *>(a.ws + a.wsl.row_scale);
    b.Rpad = round_up(a.pool.max_rank, kRankPad);
    b.y = static_cast<uint16_t *>(a.y);
    b.part = reinterpret_cast<float *>(a.ws + a.wsl.part);
    b.sync = reinterpret_cast<int *>(a.ws + a.wsl.sync);
    const dim3 grid(round_up(b.tiles_m * b.tiles_n * b.ks, kXcds));
    // Adapters in 8-bit blocks, and pools that hold none but ranks that are no multiples of 8: a wave has no plain steps.
    // Without the code for these, and with what is stored of a block behind its last step, as the loads of the next step are
    // waited for anyway, calls of one prompt of 389 rows in one kernel for all / so: rank 5 4096 x 4096 42.3 / 40.6 us, rank 36
    // 48.7 / 46.9, twice 4096 x 14336 191 / 187, rank 16 in 8-bit blocks 42.9 / 41.6, 151 / 148; 14336 x 4096 90.3 / 89.7.
    const bool gather = a.has_pool && (a.pool.q8 || (a.n_loaded > 0 && a.pool.n_odd_ranks == a.n_loaded));
    auto launch = [&](auto wfmt, auto ma) -> int {
        constexpr int WFMT = decltype(wfmt)::value, MA = decltype(ma)::value, lds = Band<WFMT, MA>::kBytes;
        auto go = [&](auto gather_c) -> int {
            constexpr bool kGather = decltype(gather_c)::value;
            static bool attr_done = false;
            if (!attr_done) {
                ELORA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&lora_band_kernel<WFMT, MA, kGather>), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
                attr_done = true;
            }
            hipLaunchKernelGGL((lora_band_kernel<WFMT, MA, kGather>), grid, dim3(kThreads), lds, stream, b, a.pool, a.has_pool ? 1 : 0);
            ELORA_HIP_TRY(hipGetLastError());
            return ELORA_OK;
        };
        return gather ? go(std::true_type{}) : go(std::false_type{});
    };
    auto with_rows = [&](auto wfmt) -> int {
        switch (s.ma) {
        case 1: return launch(wfmt, ic<1>{});
        case 2: return launch(wfmt, ic<2>{});
        case 3: return launch(wfmt, ic<3>{});
        case 4: return launch(wfmt, ic<4>{});
        case 5: return launch(wfmt, ic<5>{});
        case 6: return launch(wfmt, ic<6>{});
        default: return launch(wfmt, ic<7>{});
        }
    };
    profile_mark_begin(stream);
    int rc;
    if (a.wfmt == ELORA_W_SAME || s.copied) rc = with_rows(ic<ELORA_W_SAME>{});
    else if (a.wfmt == ELORA_W_INT8_G32) rc = with_rows(ic<ELORA_W_INT8_G32>{});
    else rc = with_rows(ic<ELORA_W_INT4_G32>{});
    if (rc == ELORA_OK) profile_mark_end(stream);
    return rc;
}
