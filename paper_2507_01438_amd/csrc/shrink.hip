// Route and shrink of the GEMM path.
//   route   per row: validated pool slot and scale (Sec. 3.4: each request names its adapter), and the list of the rows
//           that sit in short runs of equal adapters
//   shrink  V[t, :] = bf16(s_t * A_i x_t) for every row (or A_i x_t whole, as the sum of three bf16), with the rows grouped
//           by adapter inside each 32-row tile ("u-batches", Sec. 3.4 / 4.3: rows that share an adapter are computed
//           together): one masked MFMA pass per run of equal adapters; the rows of runs shorter than 8 are computed one
//           by one with plain FMAs, in the same launch or, where there may be many of them, in one of their own
#include "gemm_common.h"

#include <algorithm>

using namespace elora;

namespace {

constexpr int kShrinkRows = 32;
constexpr int kWaves = 4, kThreads = kWaves * 64;
constexpr int kMaxSlices = 4;  // K-slices per tile
constexpr int kSpan = 64;      // K elements a wave takes at a time: one whole cache line of every row
constexpr int kShortRun = 8;

// ---- route: one thread per row; a block's 256 rows are eight whole tiles of the shrink -------------------------------
constexpr int kRouteThreads = 256;
static_assert(kRouteThreads % kShrinkRows == 0, "whole tiles");

__device__ __forceinline__ void route_rows(const RouteView &route, const ShrinkArgs &s, int block)
{
    const int tid = threadIdx.x, lane = tid & 63, t = block * kRouteThreads + tid;
    for (int p = 0; p < s.n; ++p) {
        const ShrinkProj &pr = s.proj[p];
        RowRoute r{-1, 0, 0.0f};
        if (t < s.T) {
            r = resolve_row(t, route, pr.pool, true);
            pr.row_slot[t] = r.slot;
            pr.row_scale[t] = r.scale;
        }
        // the run of equal slots around this row, cut at the tile's ends (a half-wave is a tile); rows past the end of the
        // batch belong to nobody
        const int slot = t < s.T ? r.slot : INT32_MIN;
        const int before = __shfl_up(slot, 1);
        const uint64_t starts = __ballot((lane & 31) == 0 || slot != before);  // first rows of runs
        const uint32_t half = (uint32_t)(starts >> (lane & 32));
        const int q = lane & 31;
        const uint32_t upto = half & (0xffffffffu >> (31 - q)), after = q == 31 ? 0u : half & (0xfffffffeu << q);
        const int lo = 31 - __builtin_clz(upto), hi = after ? __builtin_ctz(after) : 32;
        const bool is_short = t < s.T && hi - lo < kShortRun;
        const uint64_t mk = __ballot(is_short);
        if (mk != 0) {
            int base = 0;
            if (lane == 0) base = atomicAdd(&pr.sync[kSyncShortRows], (int)__popcll(mk));
            base = __shfl(base, 0);
            if (is_short) pr.short_rows[base + (int)__popcll(mk & ((1ull << lane) - 1))] = t;
        }
    }
}

__global__ __launch_bounds__(kRouteThreads) void route_kernel(RouteView route, ShrinkArgs s) { route_rows(route, s, (int)blockIdx.x); }

// ---- rows of short runs (any rank), one by one: 16 rank entries of a row per call, four of them per wave (8-bit blocks: two at a time) --
// Bound by latency and by what a compute unit takes in: a wave takes four rows of A_i, so that x_t is read four times per
// piece, with 40 loads of 16 bytes per lane under way.  (150 rows of ranks 8 to 64, K = 4096: a whole row per workgroup on half as many
// workgroups as rows 35 us, pieces of 16 entries on one workgroup per row 24.  Against two rows of A_i at a time, x_t read
// eight times, 24 loads: gate + up of those rows 182 -> 166 us, down 93 -> 89, 600 rows of an adapter of rank 16 each 4096 x 4096
// 88 -> 78, 1800 rows of rank 32 6336 x 2048 253 -> 224.)
constexpr int kRowPiece = 16;
// Rows in short runs, as far as the host can tell, from which they are a launch of their own.  With an adapter per row, all in
// the one launch / so, calls with 512 columns of W and d_in = 4096: 300 rows of rank 16 36 / 42.5 us, 512 42 / 49.5, 1000 63 /
// 71, 2000 108 / 112, 4000 176 / 180; of ranks 8 to 64 512 rows 62 / 68, 2000 163 / 166, 4000 315 / 288.  With one adapter the
// second launch costs 2 to 3 us.  (The line was drawn when a wave took two rows of A_i and 512 rows were 89 / 84 us, 2000 243 /
// 203, 4000 of rank 16 389 / 241: what it still buys are the largest batches of mixed rank.)
constexpr int kRowsApart = 512;
// One wave: rank entries j0 .. j0 + 3 of row t (rows of A_i past the rank repeat the last one).  Two sets of loads take turns, 20
// loads of 16 bytes per lane each; x_t is read once for the four.  Every four rank entries start their walk through K at a
// different place, since rows of A_i lie a multiple of the memory channels' pitch apart: at a place that depends on the entry alone, so
// that a row's results do not depend on where in the batch it stands.
__device__ __forceinline__ void shrink_four(const uint16_t *__restrict__ A, const uint16_t *__restrict__ xt, int K, int j0, int rank, int lane, float v[4])
{
    constexpr int NL = 4;
    const int pieces = K >> 3, chunks = (pieces + 63) >> 6, rounds = (chunks + NL - 1) / NL;  // 16-byte pieces; 64 of them; NL chunks
    const int rot = chunks > 2 * NL ? (int)((unsigned)(j0 >> 2) * 5u % (unsigned)chunks) : 0;
    const bool ragged = (pieces & 63) != 0 || chunks % NL != 0;
    const uint16_t *row[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) row[r] = A + (size_t)min(j0 + r, rank - 1) * K;
    u32x4 x0[NL], a0[NL][4], x1[NL], a1[NL][4];
    auto piece_of = [&](int round, int i, bool &in) __attribute__((always_inline)) {
        int c = round * NL + i;
        in = c < chunks;
        c += rot;
        if (c >= chunks) c -= chunks;
        const int p = c * 64 + lane;
        in = in && p < pieces;
        return in ? p : 0;
    };
    auto load = [&](int round, u32x4(&x)[NL], u32x4(&a)[NL][4]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            bool in;
            const size_t off = (size_t)piece_of(round, i, in) * 8;
            x[i] = *reinterpret_cast<const u32x4 *>(xt + off);
#pragma unroll
            for (int r = 0; r < 4; ++r) a[i][r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(row[r] + off));
        }
    };
    float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto dot = [&](int round, u32x4(&x)[NL], u32x4(&a)[NL][4]) __attribute__((always_inline)) {
        if (ragged) {
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                bool in;
                (void)piece_of(round, i, in);
                if (!in) {
                    x[i] = u32x4{0, 0, 0, 0};
#pragma unroll
                    for (int r = 0; r < 4; ++r) a[i][r] = u32x4{0, 0, 0, 0};
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NL; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t aw = a[i][r][q], xw = x[i][q];
                    sum[r] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(elora_bf16x2, aw), __builtin_bit_cast(elora_bf16x2, xw), sum[r], false);
                }
    };
    load(0, x0, a0);
#pragma unroll 1
    for (int round = 0; round < rounds; round += 2) {
        if (round + 1 < rounds) load(round + 1, x1, a1);
        dot(round, x0, a0);
        if (round + 1 < rounds) {
            if (round + 2 < rounds) load(round + 2, x0, a0);
            dot(round + 1, x1, a1);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = wave_sum(sum[r]);
}

template <bool kQ8>
__device__ __forceinline__ void shrink_row_piece(const ShrinkArgs &s, const ShrinkProj &pr, int t, int first, int end)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), K = s.K;
    const int slot = pr.row_slot[t];
    const int rank = slot >= 0 ? pr.pool.meta[slot].rank : 0;
    const float sc = slot >= 0 && !pr.V_rest ? pr.row_scale[t] : 1.0f;
    const size_t at = (size_t)t * pr.Rpad;
    auto put = [&](int j, float v0, float v1) __attribute__((always_inline)) {  // two entries of the row, final
        auto store = [&](uint16_t *to, uint16_t lo, uint16_t hi) { *reinterpret_cast<uint32_t *>(to + at + j) = lo | ((uint32_t)hi << 16); };
        if (pr.V_rest) {
            uint16_t p0[3], p1[3];
            split_bf16(v0, p0);
            split_bf16(v1, p1);
            store(pr.V, p0[0], p1[0]);
            store(pr.V_rest, p0[1], p1[1]);
            store(pr.V_rest + (size_t)s.T * pr.Rpad, p0[2], p1[2]);
        } else {
            store(pr.V, f32_to_bf16(v0), f32_to_bf16(v1));
        }
    };
    if constexpr (kQ8) {
        for (int j0 = first + 2 * wave; j0 < first + kRowPiece; j0 += 2 * kWaves) {
            const bool two = j0 + 1 < rank;
            float a0 = 0.0f, a1 = 0.0f;
            if (j0 < rank) {
                const int j1 = two ? j0 + 1 : j0;
                const char *Ac = slot_A(pr.pool, slot);
                const uint16_t *As = slot_A_scales(pr.pool, slot);
                shrink_pair_q8(Ac + (size_t)j0 * K, Ac + (size_t)j1 * K, As + (((size_t)j0 * K) >> 5), As + (((size_t)j1 * K) >> 5),
                               s.x + (size_t)t * K, K, lane, a0, a1);
            }
            if (lane == 0) put(j0, j0 < rank ? sc * a0 : 0.0f, two ? sc * a1 : 0.0f);
        }
    } else {
        const int j0 = first + 4 * wave;
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (j0 < rank) shrink_four(reinterpret_cast<const uint16_t *>(slot_A(pr.pool, slot)), s.x + (size_t)t * K, K, j0, rank, lane, v);
        if (lane == 0) {
            put(j0, j0 < rank ? sc * v[0] : 0.0f, j0 + 1 < rank ? sc * v[1] : 0.0f);
            put(j0 + 2, j0 + 2 < rank ? sc * v[2] : 0.0f, j0 + 3 < rank ? sc * v[3] : 0.0f);
        }
    }
    for (int j = first + kRowPiece + 2 * tid; j < end; j += 2 * kThreads) put(j, 0.0f, 0.0f);
}

// The short rows' pieces, shared by `wgs` workgroups.  Where the pieces are no more than the workgroups, those of a row are
// side by side (a prompt whose last tile has 5 rows, K = 14336: 14.7 us, all first pieces and then all second ones 17.2).
// Else all first pieces come first: pieces beyond most rows' ranks are nothing but zeros, and fall to all workgroups alike,
// at the end.  (With 4 pieces always, and to a workgroup the same one of every row: 1846 rows of an adapter of rank 16 each,
// K = 6336, the call 297 us, so 185; 150 rows of ranks 8 to 64, K = 14336 44 and 37.)
template <bool kQ8>
__device__ __forceinline__ void shrink_rows(const ShrinkArgs &s, const ShrinkProj &pr, int n_short, int first, int wgs)
{
    const int pieces = (pr.pool.max_rank + kRowPiece - 1) / kRowPiece, items = n_short * pieces;
    for (int i = first; i < items; i += wgs) {
        const int by = items <= wgs ? pieces : n_short, hi = i / by, lo = i - hi * by;
        const int r = items <= wgs ? hi : lo, piece = items <= wgs ? lo : hi;
        // (the last piece a rank can have takes the zeros up to the end of the padded row)
        shrink_row_piece<kQ8>(s, pr, pr.short_rows[r], piece * kRowPiece, piece + 1 < pieces ? (piece + 1) * kRowPiece : pr.Rpad);
    }
}

// Many rows in short runs: a launch of their own, without LDS, so that a compute unit holds the two workgroups that the
// registers of four rows of A_i leave room for, where the rings of 64 rank entries leave one.  (Two rows of A_i at a time and
// four workgroups / so: 2000 rows of rank 64, d_in = 4096, 250 / 244 us, 600 of d_in = 14336 230 / 225, of rank 16 96 / 93,
// 4000 of ranks 8 to 64 296 / 288.  In the tiles' launch, where prompts may be all there is: within 1 % of each other for
// prompts of 389 to 7871 rows, rank 16 to 64, and 300 single rows of rank 64 55.4 / 54.5.)
template <bool kQ8>
__global__ __launch_bounds__(kThreads) void shrink_rows_kernel(ShrinkArgs s)
{
    const ShrinkProj &pr = s.proj[blockIdx.x % s.n];
    shrink_rows<kQ8>(s, pr, pr.sync[kSyncShortRows], (int)(blockIdx.x / s.n), (int)(gridDim.x / s.n));
}

// ---- a 32-row tile and one K-slice of it ---------------------------------------------------------------------------------
// Bound by how fast a compute unit takes in x and A_i.  Rows of x and of A_i travel global -> LDS in whole cache lines
// (direct loads) through a ring that every wave has to itself: a wave takes spans of 64 elements of K in turn, and no
// barrier is needed before a run's sums are added up over the waves.  (As matrix-core operands straight into registers a
// load touches half a line of each of 16 rows, and a compute unit took in 13 GB/s.)  Three quarters of the launch's time at
// 7871 rows x 14336 is x from memory; before / now: 153 / 71 us there, two projections of 4096 67 / 32, a prompt of 389
// rows 25 / 9 (d_in = 4096) and 60 / 18 (14336).  A tile is cut into
// K-slices until the launch has enough workgroups (the rule is in shrink_args); the slices' sums meet in memory (fp32), and the
// last workgroup of a tile to arrive adds them in slice order.  A tile and slice is two workgroups, which take its passes (a
// long run and as many rank entries as the ring holds) in turn: where two prompts meet in a tile, one workgroup going over x
// twice ended when the other tiles had been done for half the launch's time.  (With all passes of a run in one workgroup, the
// call with 512 columns: 7871 rows in prompts of rank 256 181 us, so 172, 400 rows 53 and 45.6, 7871 rows in 200 prompts of
// rank 32, d_in = 14336, 312 and 305.)
template <bool kQ8, int NCB>
struct Ring {
    static constexpr int kXBytes = kShrinkRows * kSpan * 2;
    static constexpr int kABytes = NCB * 16 * kSpan * (kQ8 ? 1 : 2);
    static constexpr int kScaleBytes = kQ8 ? 256 : 0;                 // one word (two fp16 scales) per row of A_i
    static constexpr int kStage = kXBytes + kABytes + kScaleBytes;
    static constexpr int kDepth = 2;  // (64 KiB at 32 rank entries: two workgroups per compute unit; 4 deep with one was no faster)
    static constexpr int kXLoads = kXBytes / 1024, kALoads = kABytes / 1024, kLoads = kXLoads + kALoads + (kQ8 ? 1 : 0);
    static constexpr int kRed = kWaves * kShrinkRows * (NCB * 16 + 4) * 4;  // the waves' sums of a run, in the same place
    static constexpr int kBytes = kWaves * kDepth * kStage > kRed ? kWaves * kDepth * kStage : kRed;
};
// The runs of equal slots among 32 rows (lane l and l + 32: row l's slot): a mask of the rows a run starts at.
__device__ __forceinline__ uint32_t run_starts(int slot, int lane)
{
    const int before = __shfl_up(slot, 1);
    return (uint32_t)__ballot((lane & 31) == 0 || slot != before);
}
__device__ __forceinline__ int run_end(uint32_t starts, int start)
{
    const uint32_t after = start == 31 ? 0u : starts & (0xfffffffeu << start);
    return after ? __builtin_ctz(after) : 32;
}

template <bool kQ8, int NCB>
__device__ __forceinline__ void shrink_tile(const ShrinkArgs &s, const ShrinkProj &pr, int tile, int slice, int part_q, int &s_last, unsigned char *ring)
{
    typedef Ring<kQ8, NCB> R;
    constexpr int kCols = NCB * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int T = s.T, K = s.K, Rpad = pr.Rpad;
    const int r0 = tile * kShrinkRows;
    float(*const s_red)[kShrinkRows][kCols + 4] = reinterpret_cast<float(*)[kShrinkRows][kCols + 4]>(ring);
    // spans [c0, c1) of the slice; this wave takes number wave, wave + 4, ... of them, counted from a place that differs
    // from tile to tile (rows of x lie a multiple of the memory channels' pitch apart: walking side by side the workgroups
    // would all ask the same few channels at a time)
    const unsigned n_spans = (unsigned)K / kSpan;
    const int c0 = (int)(n_spans * (unsigned)slice / (unsigned)s.ks), n_slice = (int)(n_spans * (unsigned)(slice + 1) / (unsigned)s.ks) - c0;
    const int n_mine = wave < n_slice ? (n_slice - wave + kWaves - 1) / kWaves : 0;
    const int turn = (int)((unsigned)(tile * 5) % (unsigned)n_slice);
    unsigned char *const mine = ring + wave * R::kDepth * R::kStage;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)mine;
    // a load moves 8 rows x 128 bytes: lane = (row, place), place = chunk ^ (row / 2) % 8, so that the 16-byte reads of 16
    // rows hit all banks.  Rows past the batch repeat the last one; what they give is dropped.
    const char *const xbase = reinterpret_cast<const char *>(s.x + (size_t)r0 * K);
    uint32_t xoff[R::kXLoads];
#pragma unroll
    for (int i = 0; i < R::kXLoads; ++i) {
        const int row = 8 * i + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
        xoff[i] = (uint32_t)(((size_t)(min(r0 + row, T - 1) - r0) * K + chunk * 8) * 2);
    }
    auto span_k = [&](int n) {  // first element of the wave's n-th span
        int c = wave + n * kWaves + turn;
        if (c >= n_slice) c -= n_slice;
        return (size_t)(c0 + c) * kSpan;
    };
    auto issue_x = [&](int n) __attribute__((always_inline)) {
        const size_t k = span_k(n);
        const uint32_t lds = lds0 + (uint32_t)(n % R::kDepth) * R::kStage;
#pragma unroll
        for (int i = 0; i < R::kXLoads; ++i) dma16(lds + i * 1024, xbase + k * 2, xoff[i]);
    };
    // (x does not depend on the routes: its first span is on its way while slots and ranks are fetched)
    if (n_mine > 0) issue_x(0);
    const int my_row = r0 + (lane & 31);
    const int slot_v = my_row < T ? pr.row_slot[my_row] : INT32_MIN;
    const float scale_v = my_row < T && !pr.V_rest ? pr.row_scale[my_row] : 1.0f;
    const int rank_v = slot_v >= 0 ? pr.pool.meta[slot_v].rank : 0;
    const uint32_t starts = run_starts(slot_v, lane);
    const int swz = (m >> 1) & 7;  // (rows 16 b + m: the same for every block b)

    // four rank entries of a row, final; those past the rank are zero whatever the sums and the scale are (an infinite scale
    // times zero would be NaN)
    auto put = [&](int r, int c, floatx4 v, int rank, float scale) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = c + i < rank ? v[i] * scale : 0.0f;
        const size_t at = (size_t)(r0 + r) * Rpad + c;
        auto store = [&](uint16_t *to, uint16_t h0, uint16_t h1, uint16_t h2, uint16_t h3) {
            *reinterpret_cast<uint64_t *>(to + at) = (uint64_t)h0 | ((uint64_t)h1 << 16) | ((uint64_t)h2 << 32) | ((uint64_t)h3 << 48);
        };
        if (pr.V_rest) {
            uint16_t p[4][3];
#pragma unroll
            for (int i = 0; i < 4; ++i) split_bf16(v[i], p[i]);
            store(pr.V, p[0][0], p[1][0], p[2][0], p[3][0]);
            store(pr.V_rest, p[0][1], p[1][1], p[2][1], p[3][1]);
            store(pr.V_rest + (size_t)T * Rpad, p[0][2], p[1][2], p[2][2], p[3][2]);
        } else {
            store(pr.V, f32_to_bf16(v[0]), f32_to_bf16(v[1]), f32_to_bf16(v[2]), f32_to_bf16(v[3]));
        }
    };
    // sums of slice k: [row][entry], written through to memory and read past the caches' first level (the workgroups of a
    // tile run on one XCD as a rule, but nothing depends on it)
    constexpr int kCoherent = 16;  // sc1
    auto rsrc = __builtin_amdgcn_make_buffer_rsrc(pr.part + (size_t)tile * s.ks * kShrinkRows * Rpad, 0, s.ks * kShrinkRows * Rpad * 4, 0x00020000);
    auto part_at = [&](int k, int r, int c) { return ((k * kShrinkRows + r) * Rpad + c) * 4; };

    bool x_under_way = true;
    int turns = 0;  // passes over long runs with an adapter met so far: the two parts take them in turn
    for (int start = 0; start < kShrinkRows;) {
        const int slot = __builtin_amdgcn_readlane(slot_v, start), end = run_end(starts, start);
        const bool is_long = slot >= 0 && end - start >= kShortRun;
        if (is_long) {
            const int rank = __builtin_amdgcn_readlane(rank_v, start);
            const char *const A = slot_A(pr.pool, slot);
            const char *const As = reinterpret_cast<const char *>(slot_A_scales(pr.pool, slot));  // (8-bit blocks)
            for (int j0 = 0; j0 < rank; j0 += kCols) {
                if ((turns++ & 1) != part_q) continue;
                // rows of A_i past the rank repeat the last one; what they give is dropped
                uint32_t aoff[R::kALoads], soff = 0;
#pragma unroll
                for (int i = 0; i < R::kALoads; ++i) {
                    if constexpr (kQ8) {  // 16 rows x 64 bytes: place = chunk ^ (row / 4) % 4
                        const int row = 16 * i + (lane >> 2), chunk = (lane & 3) ^ ((row >> 2) & 3);
                        aoff[i] = (uint32_t)((size_t)min(j0 + row, rank - 1) * K + chunk * 16);
                    } else {
                        const int row = 8 * i + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
                        aoff[i] = (uint32_t)(((size_t)min(j0 + row, rank - 1) * K + chunk * 8) * 2);
                    }
                }
                if constexpr (kQ8) soff = (uint32_t)((size_t)min(j0 + (lane & (kCols - 1)), rank - 1) * (K >> 5) * 2);
                auto issue_a = [&](int n) __attribute__((always_inline)) {
                    const size_t k = span_k(n);
                    const uint32_t lds = lds0 + (uint32_t)(n % R::kDepth) * R::kStage + R::kXBytes;
#pragma unroll
                    for (int i = 0; i < R::kALoads; ++i) dma16(lds + i * 1024, A + k * (kQ8 ? 1 : 2), aoff[i]);
                    if constexpr (kQ8) dma4(lds + R::kABytes, As + (k >> 5) * 2, soff);
                };
                floatx4 acc[2][NCB];
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < NCB; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (n_mine > 0) {
                    if (!x_under_way) issue_x(0);
                    issue_a(0);
                }
                x_under_way = false;
                for (int n = 0; n < n_mine; ++n) {
                    // (the reads of the stage that the next loads go to, one turn ago, are over)
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    if (n + 1 < n_mine) {
                        issue_x(n + 1);
                        issue_a(n + 1);
                        wait_loads<R::kLoads>();
                    } else {
                        wait_loads<0>();
                    }
                    const unsigned char *const st = mine + (n % R::kDepth) * R::kStage;
#pragma unroll
                    for (int k = 0; k < kSpan / 32; ++k) {
                        bf16x8 xa[2], ab[NCB];
                        const int place = ((k * 4 + g) ^ swz) * 16;
#pragma unroll
                        for (int a = 0; a < 2; ++a) xa[a] = *reinterpret_cast<const bf16x8 *>(st + (a * 16 + m) * 128 + place);
#pragma unroll
                        for (int b = 0; b < NCB; ++b) {
                            if constexpr (kQ8) {
                                // chunk of 16 codes 2 k + g / 2, its half g % 2
                                const unsigned char *row = st + R::kXBytes + (b * 16 + m) * 64;
                                const u32x2 codes = *reinterpret_cast<const u32x2 *>(row + (((2 * k + (g >> 1)) ^ ((m >> 2) & 3)) * 16) + (g & 1) * 8);
                                const uint16_t sc = *reinterpret_cast<const uint16_t *>(st + R::kXBytes + R::kABytes + (b * 16 + m) * 4 + k * 2);
                                ab[b] = __builtin_bit_cast(bf16x8, q8_to_bf16x8(codes, fp16_to_f32(sc)));
                            } else {
                                ab[b] = *reinterpret_cast<const bf16x8 *>(st + R::kXBytes + (b * 16 + m) * 128 + place);
                            }
                        }
#pragma unroll
                        for (int a = 0; a < 2; ++a)
#pragma unroll
                            for (int b = 0; b < NCB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ab[b], xa[a], acc[a][b], 0, 0, 0);
                    }
                }
                __syncthreads();  // every wave is done with its ring
                // MFMA rows = rank rows j (A-operand), columns = batch rows (B-operand): lane holds batch row (lane % 16), rank
                // rows (lane / 16) * 4 + 0..3
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < NCB; ++b) *reinterpret_cast<floatx4 *>(&s_red[wave][a * 16 + m][b * 16 + g * 4]) = acc[a][b];
                __syncthreads();
                for (int e = tid; e < kShrinkRows * (kCols / 4); e += kThreads) {
                    const int r = e / (kCols / 4), c4 = (e % (kCols / 4)) * 4;
                    const float scale = __shfl(scale_v, r & 31);
                    if (r < start || r >= end) continue;
                    floatx4 v = *reinterpret_cast<const floatx4 *>(&s_red[0][r][c4]);
#pragma unroll
                    for (int w = 1; w < kWaves; ++w) v += *reinterpret_cast<const floatx4 *>(&s_red[w][r][c4]);
                    if (s.ks == 1) put(r, j0 + c4, v, rank, scale);
                    else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrc, part_at(slice, r, j0 + c4), 0, kCoherent);
                }
                __syncthreads();
            }
            // zeros between the last pass and the end of the padded row
            if (slice == 0 && part_q == 0) {
                const int done = (rank + kCols - 1) / kCols * kCols, left = (Rpad - done) / 4;
                if (left > 0)
                    for (int e = tid; e < (end - start) * left; e += kThreads)
                        put(start + e / left, done + (e % left) * 4, floatx4{0.f, 0.f, 0.f, 0.f}, 0, 1.0f);
            }
        } else if (slot == -1 && end - start >= kShortRun && slice == 0 && part_q == 0) {
            for (int e = tid; e < (end - start) * (Rpad / 4); e += kThreads)
                put(start + e / (Rpad / 4), (e % (Rpad / 4)) * 4, floatx4{0.f, 0.f, 0.f, 0.f}, 0, 1.0f);
        }
        start = end;
    }
    // (loads of x that no run of this tile waited for: they land before the ring is used again)
    if (x_under_way) wait_loads<0>();
    if (s.ks == 1) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's sums have reached memory
    __syncthreads();
    if (tid == 0) {
        const int before = __hip_atomic_fetch_add(&pr.sync[kSyncTiles + tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = before == 2 * s.ks - 1;
        if (s_last) __hip_atomic_store(&pr.sync[kSyncTiles + tile], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!s_last) return;
    for (int start = 0; start < kShrinkRows;) {
        const int slot = __builtin_amdgcn_readlane(slot_v, start), end = run_end(starts, start);
        if (slot >= 0 && end - start >= kShortRun) {
            const int rank = __builtin_amdgcn_readlane(rank_v, start), cols = (rank + kCols - 1) / kCols * (kCols / 4);
            for (int e0 = 0; e0 < (end - start) * cols; e0 += kThreads) {
                const int e = e0 + tid, r = min(start + e / cols, end - 1), c = (e % cols) * 4;
                const float scale = __shfl(scale_v, r);
                u32x4 w[kMaxSlices];
#pragma unroll
                for (int k = 0; k < kMaxSlices; ++k) w[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, part_at(min(k, s.ks - 1), r, c), 0, kCoherent);
                floatx4 v = __builtin_bit_cast(floatx4, w[0]);
#pragma unroll
                for (int k = 1; k < kMaxSlices; ++k)
                    if (k < s.ks) v += __builtin_bit_cast(floatx4, w[k]);
                if (e < (end - start) * cols) put(r, c, v, rank, scale);
            }
        }
        start = end;
    }
}

// A projection's workgroups: consecutive tiles per XCD, the slices of a tile next to each other on one XCD.
template <bool kQ8, int NCB>
__device__ __forceinline__ void shrink_workgroup(const ShrinkArgs &s, int wg)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char ring[];  // Ring<kQ8, NCB>::kBytes
    __shared__ int s_last;
    // workgroup wg: XCD wg % 8; on an XCD the projections take turns, so that those that read the same rows of x run side by
    // side and all but the first find them in its L2
    const int xcd = wg % kXcds, j = wg / kXcds;
    const ShrinkProj &pr = s.proj[j % s.n];
    const int seq = j / s.n;
    const int tiles_per_xcd = (s.n_tiles + kXcds - 1) / kXcds;
    // (second parts first: all but the few that have something to do end at once and make room)
    const int units = tiles_per_xcd * s.ks, part_q = seq < units ? 1 : 0, u = seq - (part_q ? 0 : units);
    const int tile = xcd * tiles_per_xcd + u / s.ks;
    const int n_short = pr.sync[kSyncShortRows];
    if (u < units && tile < s.n_tiles) shrink_tile<kQ8, NCB>(s, pr, tile, u % s.ks, part_q, s_last, ring);
    // the rows of short runs are shared by all workgroups (a few workgroups of their own would each wait for a ring's worth of LDS)
    if (!s.rows_apart) shrink_rows<kQ8>(s, pr, n_short, seq * kXcds + xcd, s.wgs_per_xcd * kXcds);
}
int shrink_grid(const ShrinkArgs &s) { return s.wgs_per_xcd * kXcds * s.n; }

template <bool kQ8, int NCB>
__global__ __launch_bounds__(kThreads) void sgmv_shrink_kernel(ShrinkArgs s)
{
    shrink_workgroup<kQ8, NCB>(s, (int)blockIdx.x);
}

// ---- the bf16 copy of a 4-bit or 8-bit W -------------------------------------------------------------------------------
// Many rows: W is converted to bf16 once per call, into the workspace, and the bf16 GEMM runs on the copy.
// One thread per 8 weights (4 or 8 bytes of codes in, 16 bytes out; four threads share a group's fp16 scale).
// 8-bit: w = scale * code; 4-bit: w = fma(code, scale, -8 scale); exact in fp32, rounded once.
template <int WFMT>
__device__ __forceinline__ void w_dequant_piece(size_t i, size_t n_pieces, const uint32_t *__restrict__ codes,
                                                const uint16_t *__restrict__ scales, u32x4 *__restrict__ out)
{
    if (i >= n_pieces) return;
    const float sc = fp16_to_f32(scales[i >> 2]);
    if constexpr (WFMT == ELORA_W_INT8_G32) {
        out[i] = q8_to_bf16x8(reinterpret_cast<const u32x2 *>(codes)[i], sc);
    } else {
        out[i] = w4_to_bf16x8(codes[i], sc);
    }
}

// The routes and the copy in one launch (the routes' few workgroups first): they do not depend on each other, and neither
// needs LDS.  (With the shrink the copy would share the ring's LDS, which leaves a compute unit one workgroup.)
template <int WFMT>
__global__ __launch_bounds__(kRouteThreads) void route_w_dequant_kernel(RouteView route, ShrinkArgs s, int n_route, size_t n_pieces, const uint32_t *__restrict__ codes,
                                                                        const uint16_t *__restrict__ scales, u32x4 *__restrict__ out)
{
    if ((int)blockIdx.x < n_route) {
        route_rows(route, s, (int)blockIdx.x);
        return;
    }
    w_dequant_piece<WFMT>((size_t)(blockIdx.x - n_route) * kRouteThreads + threadIdx.x, n_pieces, codes, scales, out);
}

template <typename F>
auto with_cols(const ShrinkArgs &s, F &&f)  // f(8-bit blocks, MFMA column blocks per pass)
{
    int most = 1;
    for (int p = 0; p < s.n; ++p) most = s.proj[p].pool.max_rank > most ? s.proj[p].pool.max_rank : most;
    auto cols = [&](auto q8) {
        if (most <= 16) return f(q8, ic<1>{});
        if (most <= 32 || s.by_row) return f(q8, ic<2>{});
        return f(q8, ic<4>{});
    };
    return s.proj[0].pool.q8 ? cols(std::true_type{}) : cols(std::false_type{});
}

}  // namespace

// (how many rows may sit in short runs: every row that has an index of its own, some at the ends of a segment)
bool elora::shrink_rows_apart(int T, bool indices, int n_segments) { return std::min((long long)T, indices ? (long long)T : 3ll * n_segments) >= kRowsApart; }

void elora::shrink_args(ShrinkArgs &s, const LinearArgs *a, int n, const bool *whole)
{
    s.n = n;
    s.T = a[0].T;
    s.K = a[0].K;
    s.x = static_cast<const uint16_t *>(a[0].x);
    s.n_tiles = (s.T + kShrinkRows - 1) / kShrinkRows;
    // K-slices, up to 4 (every further one adds to the time at the end, when the last workgroup of a tile reads all sums):
    // as many as leave a projection at most one workgroup per compute unit, or two while a slice is still 4096 elements or
    // more (7871 rows: d_in = 14336 76 -> 71 us with two, d_in = 4096 32 -> 36), with at least two spans per wave and slice,
    // and within the room for the slices' sums and the counters.
    auto room_for = [&](int ks) {
        for (int p = 0; p < n; ++p)
            if ((size_t)s.n_tiles * kShrinkRows * round_up(a[p].pool.max_rank, kRankPad) * sizeof(float) * ks > a[p].wsl.part_bytes) return false;
        return true;
    };
    s.ks = 1;
    while (s.ks < kMaxSlices && s.n_tiles * (s.ks + 1) <= (s.K / (s.ks + 1) >= 4096 ? 512 : 256) && s.n_tiles <= kSyncTileCount &&
           s.K / kSpan >= (s.ks + 1) * 2 * kWaves && room_for(s.ks + 1))
        ++s.ks;
    s.rows_apart = shrink_rows_apart(s.T, a[0].route.adapter_idx != nullptr, a[0].route.n_segments);
    // Rows with an index of their own, and more adapters than an eighth of them: long runs are unlikely, and the rings of 32
    // rank entries leave a compute unit two workgroups for the rows instead of one.  With rings of 64 / so, calls with 512
    // columns: 300 rows of their own of rank 64, d_in = 2048 44.8 / 40.5 us, 4096 57 / 51.5, 8192 81 / 74.5, of rank 128 64 /
    // 55, 82.5 / 75.5, 125.5 / 122.5, 400 of rank 256, 4096, 169 / 143; if they are all of one adapter after all, rank 64 25.7
    // / 25.1, 27.6 / 26.8, 32.5 / 31, rank 128 30.9 / 31.8 (4096), rank 256 44 / 45.6.  Not where the rows are a launch of
    // their own (700 of rank 64 89.0 / 88.0 us, 256 263 / 264), nor for 8-bit blocks, whose rings of 64 fit twice (300 of rank
    // 64 and 256 within 1 %).  For longer rows it was measured on 150 rows of ranks 8 to 64, d_in = 14336 (88.8 us with one
    // workgroup, 93.4 with two); 300 rows of rank 64 would gain there as well (120 / 114).
    s.by_row = a[0].route.adapter_idx != nullptr && !s.rows_apart && s.K <= 8192;
    for (int p = 0; p < n; ++p) s.by_row = s.by_row && !a[p].pool.q8 && a[p].n_loaded * 8ll > s.T;
    // (at least four workgroups per row, up to two per compute unit: the rows of short runs are shared by all of them)
    s.wgs_per_xcd = std::max((s.n_tiles + kXcds - 1) / kXcds * s.ks * 2, std::min((s.T + 1) / 2, 64));
    for (int p = 0; p < n; ++p) {
        ShrinkProj &q = s.proj[p];
        q.pool = a[p].pool;
        q.row_slot = reinterpret_cast<int32_t *>(a[p].ws + a[p].wsl.row_slot);
        q.row_scale = reinterpret_cast<float *>(a[p].ws + a[p].wsl.row_scale);
        q.short_rows = reinterpret_cast<int32_t *>(a[p].ws + a[p].wsl.short_rows);
        q.V = reinterpret_cast<uint16_t *>(a[p].ws + a[p].wsl.v);
        q.V_rest = whole[p] ? reinterpret_cast<uint16_t *>(a[p].ws + a[p].wsl.v_rest) : nullptr;
        q.part = reinterpret_cast<float *>(a[p].ws + a[p].wsl.part);
        q.sync = reinterpret_cast<int *>(a[p].ws + a[p].wsl.sync);
        q.Rpad = round_up(a[p].pool.max_rank, kRankPad);
    }
}

int elora::launch_route(const ShrinkArgs &s, const LinearArgs *a, bool copy, hipStream_t stream)
{
    const int n_route = a[0].has_pool ? (s.T + kRouteThreads - 1) / kRouteThreads : 0;
    if (copy) {
        const size_t n_pieces = (size_t)a[0].N * (size_t)(a[0].K / 8);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3((unsigned)(n_route + (n_pieces + kRouteThreads - 1) / kRouteThreads)), dim3(kRouteThreads), 0, stream, a[0].route, s,
                               n_route, n_pieces, static_cast<const uint32_t *>(a[0].W), static_cast<const uint16_t *>(a[0].w_scales),
                               reinterpret_cast<u32x4 *>(a[0].ws + a[0].wsl.wdeq));
        };
        if (a[0].wfmt == ELORA_W_INT8_G32) go(route_w_dequant_kernel<ELORA_W_INT8_G32>);
        else go(route_w_dequant_kernel<ELORA_W_INT4_G32>);
    } else if (n_route > 0) {
        hipLaunchKernelGGL(route_kernel, dim3(n_route), dim3(kRouteThreads), 0, stream, a[0].route, s);
    }
    ELORA_HIP_TRY(hipGetLastError());
    return ELORA_OK;
}

int elora::launch_shrink(const ShrinkArgs &s, hipStream_t stream)
{
    return with_cols(s, [&](auto q8, auto ncb) -> int {
        constexpr bool Q8 = decltype(q8)::value;
        constexpr int NCB = decltype(ncb)::value, lds = Ring<Q8, NCB>::kBytes;
        static bool attr_done = false;
        if (!attr_done) {
            ELORA_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&sgmv_shrink_kernel<Q8, NCB>), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            attr_done = true;
        }
        hipLaunchKernelGGL((sgmv_shrink_kernel<Q8, NCB>), dim3(shrink_grid(s)), dim3(kThreads), lds, stream, s);
        ELORA_HIP_TRY(hipGetLastError());
        if (s.rows_apart) {
            hipLaunchKernelGGL((shrink_rows_kernel<Q8>), dim3(1024 * s.n), dim3(kThreads), 0, stream, s);
            ELORA_HIP_TRY(hipGetLastError());
        }
        return ELORA_OK;
    });
}
