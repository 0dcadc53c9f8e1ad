// The fp32 path (any shape, any rank): two launches, or one for the smallest calls (fp32_one_kernel).
//   route + shrink   per row: pool slot and scale (Sec. 3.4: each request names its adapter), v_t = A_i x_t
//   product          y_t = W x_t + s * B_i v_t, written at row t (Sec. 3.4 closing equation)
// Calls of this path are small (a model kept in fp32 to check an adapter), so what bounds them is latency: few launches, every
// load of a wave under way at once, and K split over the waves of a workgroup so that a call of a few rows still has a
// wave on most compute units.  Products and sums are fp32 throughout, on the fp32 matrix instructions.  Calls with rank-16
// adapters, three launches of plain FMAs through 64 x 64 tiles / here: 8 rows 512 x 512 67 / 7.8 us, 155 rows 1000 x 1430
// 162 / 17, 272 rows 2048 x 3000 317 / 81, 2000 rows 2048 x 2048 615 / 294, 4096 rows 4096 x 4096 4182 / 2198 (there the
// loads of a 32 x 32 tile bound it: 8 products per byte); error against 64-bit sums 4 to 11 e-7 / 1.5 to 4 e-7.
#include <algorithm>

#include "common.h"

using namespace elora;

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
struct __attribute__((packed, aligned(4))) float4_dword {  // four floats at any float's address (rows may have any length)
    float v[4];
};
__device__ __forceinline__ floatx4 load4(const float *p)
{
    const float4_dword f = *reinterpret_cast<const float4_dword *>(p);
    return floatx4{f.v[0], f.v[1], f.v[2], f.v[3]};
}
// elements k .. k + 3 of a row of K, zero past its end
__device__ __forceinline__ floatx4 load4_until(const float *row, int k, int K)
{
    floatx4 v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (k + i < K) v[i] = row[k + i];
    return v;
}

constexpr int kThreads = 512, kWaves = kThreads / 64;

// ---- route + shrink: a workgroup per row and 16 rank entries, a wave takes two of them --------------------------------------
constexpr int kPiece = 2 * kWaves;
__global__ __launch_bounds__(kThreads) void fp32_shrink_kernel(int K, const float *__restrict__ x, RouteView route, PoolView pool, int32_t *__restrict__ row_slot,
                                                               float *__restrict__ row_scale, float *__restrict__ V, int R, int t_first)
{
    const int t = t_first + (int)blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool owner = blockIdx.y == 0 && threadIdx.x == 0;  // (a bad index is counted once per row)
    const RowRoute r = resolve_row(t, route, pool, owner);
    if (owner) {
        row_slot[t] = r.slot;
        row_scale[t] = r.scale;
    }
    const int j0 = (int)blockIdx.y * kPiece + 2 * wave;
    if (r.slot < 0 || j0 >= r.rank) return;
    const bool two = j0 + 1 < r.rank;
    const float *const A0 = reinterpret_cast<const float *>(slot_A(pool, r.slot)) + (size_t)j0 * K, *const A1 = two ? A0 + K : A0, *const xt = x + (size_t)t * K;
    float s0 = 0.0f, s1 = 0.0f;
    int k = lane * 4;
    for (; k + 3 < K - 768; k += 1024) {  // four passes' loads in flight
        floatx4 a[4], b[4], c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = load4(A0 + k + i * 256);
            b[i] = load4(A1 + k + i * 256);
            c[i] = load4(xt + k + i * 256);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s0 = fmaf(a[i][q], c[i][q], s0);
                s1 = fmaf(b[i][q], c[i][q], s1);
            }
    }
#pragma unroll 4
    for (; k < K; k += 256) {
        floatx4 a, b, c;
        if (k + 3 < K) {
            a = load4(A0 + k);
            b = load4(A1 + k);
            c = load4(xt + k);
        } else {
            a = load4_until(A0, k, K);
            b = load4_until(A1, k, K);
            c = load4_until(xt, k, K);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            s0 = fmaf(a[q], c[q], s0);
            s1 = fmaf(b[q], c[q], s1);
        }
    }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    if (lane == 0) {
        V[(size_t)t * R + j0] = s0;
        if (two) V[(size_t)t * R + j0 + 1] = s1;
    }
}

// ---- product: 16 MB rows x 16 NB columns per workgroup, K split over its eight waves in turns of 16 -------------------------
// A lane takes four consecutive elements of row lane % 16 (elements 4 (lane / 16) .. + 3 of the turn's 16), straight from memory:
// the four matrix instructions of a turn multiply element i of every lane, in which order K is walked does not matter.
// The eight waves' sums meet in LDS and are added in wave order.
// One turn's loads of a wave are under way beside those that are multiplied, and it is the eight waves and the other workgroups
// of a compute unit that hide them: with one turn ahead four workgroups fit (the 32 x 32 tile with four ahead: 157 registers,
// one).  Rank-8 calls, four ahead / one, 272 rows 1000 x 3000 50 / 42 us, 2000 rows 128 x 10000 440 / 144, 2048 x 10000
// 1556 / 1336; 16 rows 2048 x 3000 13.8 / 13.2.  A launch of one 32 x 16 tile per compute unit has two turns ahead (60 rows
// 2048 x 2048 18.2 us, four 19.1).
template <int MB, int NB, int kAhead>
__global__ __launch_bounds__(kThreads, kAhead == 1 ? 8 : 1) void fp32_product_kernel(int T, int K, int N, const float *__restrict__ x, const float *__restrict__ W, PoolView pool, int has_pool,
                                                                const int32_t *__restrict__ row_slot, const float *__restrict__ row_scale,
                                                                const float *__restrict__ V, int R, float *__restrict__ y, int first_tile)
{
    constexpr int kRows = 16 * MB, kCols = 16 * NB;  // (kAhead: turns whose loads are in flight)
    __shared__ float s_sum[kWaves][kRows][kCols + 4];
    __shared__ int s_slot[kRows], s_rank[kRows];
    __shared__ float s_scale[kRows];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = lane & 15, g = lane >> 4;
    const int tiles_n = (N + kCols - 1) / kCols, tile = first_tile + (int)blockIdx.x;
    const int t0 = tile / tiles_n * kRows, n0 = tile % tiles_n * kCols;
    // rows past the end of x and W repeat the last one; what they give is never stored
    const float *xr[MB], *wr[NB];
#pragma unroll
    for (int a = 0; a < MB; ++a) xr[a] = x + (size_t)min(t0 + a * 16 + m, T - 1) * K + g * 4;
#pragma unroll
    for (int b = 0; b < NB; ++b) wr[b] = W + (size_t)min(n0 + b * 16 + m, N - 1) * K + g * 4;
    floatx4 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const floatx4 *xv, const floatx4 *wv) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[b][i], xv[a][i], acc[a][b], 0, 0, 0);
    };
    const int whole = K / 16;  // turns that need no test
    const int n_mine = wave < whole ? (whole - wave + kWaves - 1) / kWaves : 0;
    floatx4 xv[2][kAhead][MB], wv[2][kAhead][NB];
    auto fetch = [&](int to, int first) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const size_t k = (size_t)(wave + min(first + i, n_mine - 1) * kWaves) * 16;
#pragma unroll
            for (int a = 0; a < MB; ++a) xv[to][i][a] = load4(xr[a] + k);
#pragma unroll
            for (int b = 0; b < NB; ++b) wv[to][i][b] = load4(wr[b] + k);
        }
    };
    auto use = [&](int from, int first) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (first + i < n_mine) multiply(xv[from][i], wv[from][i]);
    };
    if (n_mine > 0) {
        fetch(0, 0);
        for (int n = 0; n < n_mine; n += 2 * kAhead) {
            if (n + kAhead < n_mine) fetch(1, n + kAhead);
            use(0, n);
            if (n + 2 * kAhead < n_mine) fetch(0, n + 2 * kAhead);
            if (n + kAhead < n_mine) use(1, n + kAhead);
        }
    }
    if (whole * 16 < K && wave == whole % kWaves) {  // the turn that K ends in
        floatx4 xt[MB], wt[NB];
#pragma unroll
        for (int a = 0; a < MB; ++a) xt[a] = load4_until(xr[a], whole * 16, K - g * 4);
#pragma unroll
        for (int b = 0; b < NB; ++b) wt[b] = load4_until(wr[b], whole * 16, K - g * 4);
        multiply(xt, wt);
    }
    // (one row's route per lane: asked for per output, these are two more trips to memory behind the product)
    if (tid < kRows) {
        const int t = min(t0 + tid, T - 1), slot = has_pool ? row_slot[t] : -1;
        s_slot[tid] = slot;
        s_rank[tid] = slot >= 0 ? pool.meta[slot].rank : 0;
        s_scale[tid] = slot >= 0 ? row_scale[t] : 0.0f;
    }
    // a lane holds columns 4 g .. + 3 of row m
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) *reinterpret_cast<floatx4 *>(&s_sum[wave][a * 16 + m][b * 16 + g * 4]) = acc[a][b];
    __syncthreads();
    for (int e = tid; e < kRows * kCols; e += kThreads) {
        const int rl = e / kCols, cl = e % kCols, t = t0 + rl, n = n0 + cl;
        if (t >= T || n >= N) continue;
        float sum = s_sum[0][rl][cl];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) sum += s_sum[w][rl][cl];
        const int slot = s_slot[rl], rank = s_rank[rl];
        if (slot >= 0) {
            const float *const Bn = reinterpret_cast<const float *>(slot_B(pool, slot)) + (size_t)n * rank, *const v = V + (size_t)t * R;
            float d = 0.0f;
            int q = 0;
            for (; q + 8 <= rank; q += 8) {
                const floatx4 b0 = load4(Bn + q), b1 = load4(Bn + q + 4), v0 = load4(v + q), v1 = load4(v + q + 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) d = fmaf(v0[i], b0[i], d);
#pragma unroll
                for (int i = 0; i < 4; ++i) d = fmaf(v1[i], b1[i], d);
            }
            if (q < rank) {
                float bq[8], vq[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    bq[i] = q + i < rank ? Bn[q + i] : 0.0f;
                    vq[i] = q + i < rank ? v[q + i] : 0.0f;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (q + i < rank) d = fmaf(vq[i], bq[i], d);
            }
            sum += s_scale[rl] * d;
        }
        y[(size_t)t * N + n] = sum;
    }
}

// ---- one launch: the product of a small call with the shrink in it -----------------------------------------------------------
// What bounds a small call is launches and trips to memory, so here every workgroup (16 rows x 16 columns, four waves that
// split K) forms the shrink results of its own rows: the ranks of their different adapters, one behind the other, are
// further columns of the product, 32 beside the tile's own 16, and what there is beyond 32 in further walks over K.  Every
// wave resolves the rows' routes by itself while its first loads of x and W are under way, and a thread's row of B_i is
// on its way during the walk.  Two launches / one, rank-8 calls: 8 rows 512 x 512 7.8 / 7.0 us, 3 rows 64 x 64 7.4 / 4.8, 16
// rows 300 x 2000 7.5 / 6.0, 33 rows 100 x 1000 7.5 / 4.9; see one_launch for where it ends.
constexpr int kOneTile = 16, kOneRanks = 32, kOneWaves = 4;
__global__ __launch_bounds__(64 * kOneWaves) void fp32_one_kernel(int T, int K, int N, const float *__restrict__ x, const float *__restrict__ W, PoolView pool, RouteView route,
                                                                  float *__restrict__ y)
{
    constexpr int kBlocks = kOneRanks / 16, kAhead = 2, kPitch = kOneTile + kOneRanks + 4, kEarly = 4;
    static_assert(kOneTile == 16 && kOneTile * kOneTile == 64 * kOneWaves, "an output per thread");
    __shared__ __attribute__((aligned(16))) float s_sum[kOneWaves][kOneTile][kPitch];
    __shared__ float s_v[kOneTile][kOneRanks];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = lane & 15, g = lane >> 4;
    const int tiles_n = (N + kOneTile - 1) / kOneTile;
    const int t0 = (int)blockIdx.x / tiles_n * kOneTile, n0 = (int)blockIdx.x % tiles_n * kOneTile;
    // rows past the end of x and W repeat the last one; what they give is never stored
    const int mine = min(t0 + m, T - 1);  // (the lane's row of x, and the row whose route it resolves)
    const RouteIndex ri = route_index(mine, route);
    SlotMeta meta{0, 0.0f, 0, 0};
    if (ri.idx >= 0 && ri.idx < pool.capacity) meta = pool.meta[ri.idx];
    const float given = route.scales != nullptr && ri.idx != -1 ? route.scales[ri.scale_at] : 0.0f;
    const float *const xr = x + (size_t)mine * K + g * 4, *const wr = W + (size_t)min(n0 + m, N - 1) * K + g * 4;
    const int whole = K / 16;  // turns that need no test
    const int n_mine = wave < whole ? (whole - wave + kOneWaves - 1) / kOneWaves : 0;
    auto at = [&](int turn) { return (size_t)(wave + min(turn, n_mine - 1) * kOneWaves) * 16; };
    floatx4 xv[2][kAhead], wv[2][kAhead], av[2][kAhead][kBlocks];
    auto fetch_x = [&](int to, int first) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) xv[to][i] = load4(xr + at(first + i));
    };
    auto fetch_w = [&](int to, int first) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) wv[to][i] = load4(wr + at(first + i));
    };
    if (n_mine > 0) {
        fetch_x(0, 0);
        fetch_w(0, 0);
    }
    // (a bad index is counted once per row)
    const RowRoute r = route_finish(mine, ri, meta, given, route, pool, n0 == 0 && tid < kOneTile && t0 + tid < T);
    // the different adapters of the rows: `total` ranks one behind the other, the lane's own from `off` on
    const uint64_t served = __ballot(r.slot >= 0 && lane < kOneTile);
    int total = 0, off = 0;
    for (uint64_t left = served; left != 0;) {
        const int i = (int)__builtin_ctzll(left), slot = __builtin_amdgcn_readlane(r.slot, i);
        if (r.slot == slot) off = total;
        left &= ~__ballot(r.slot == slot);
        total += __builtin_amdgcn_readlane(r.rank, i);
    }
    // the thread's output: row rl, column n, and the first entries of its row of B_i
    const int rl = tid / kOneTile, n = n0 + tid % kOneTile;
    const int my_off = __shfl(off, rl), my_rank = __shfl(r.rank, rl), my_slot = __shfl(r.slot, rl);
    const float my_scale = __shfl(r.scale, rl);
    const float *const Bn = reinterpret_cast<const float *>(slot_B(pool, max(my_slot, 0))) + (size_t)min(n, N - 1) * my_rank;
    floatx4 early[kEarly];
#pragma unroll
    for (int q = 0; q < kEarly; ++q) {
        early[q] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (my_slot >= 0 && 4 * q + 4 <= my_rank) early[q] = load4(Bn + 4 * q);
    }
    // two sums of every output, added at the end: as many products go into one as on the two launches, where eight waves split K
    // (8 rows 512 x 512, error against 64-bit sums 2.6e-7 with one sum, 1.7e-7 on the two launches)
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
    float sum = 0.0f, d = 0.0f;
    // One walk over K: `blocks` 16 ranks from first_rank on, and in the first walk the tile's own columns.
    auto walk = [&](auto with_w_c, auto blocks_c, int first_rank) __attribute__((always_inline)) {
        constexpr bool with_w = decltype(with_w_c)::value;
        constexpr int blocks = decltype(blocks_c)::value;
        const float *ar[kBlocks];
        floatx4 accv[kBlocks][2];
#pragma unroll
        for (int p = 0; p < blocks; ++p) {
            const int c = min(first_rank + p * 16 + m, total - 1);  // (those past the last repeat it, and nobody takes them)
            int slot = 0, j = 0;
            for (uint64_t left = served; left != 0;) {
                const int i = (int)__builtin_ctzll(left), s = __builtin_amdgcn_readlane(r.slot, i), begin = __builtin_amdgcn_readlane(off, i);
                if (c >= begin) {
                    slot = s;
                    j = c - begin;
                }
                left &= ~__ballot(r.slot == s);
            }
            ar[p] = reinterpret_cast<const float *>(slot_A(pool, slot)) + (size_t)j * K + g * 4;
            accv[p][0] = accv[p][1] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        auto fetch_a = [&](int to, int first) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
#pragma unroll
                for (int p = 0; p < blocks; ++p) av[to][i][p] = load4(ar[p] + at(first + i));
        };
        auto fetch = [&](int to, int first) __attribute__((always_inline)) {
            fetch_x(to, first);
            if constexpr (with_w) fetch_w(to, first);
            fetch_a(to, first);
        };
        auto multiply = [&](const floatx4 &x4, const floatx4 &w4, const floatx4 *a4) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (with_w) acc[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w4[i], x4[i], acc[i & 1], 0, 0, 0);
#pragma unroll
                for (int p = 0; p < blocks; ++p) accv[p][i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[p][i], x4[i], accv[p][i & 1], 0, 0, 0);
            }
        };
        auto use = [&](int from, int first) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < kAhead; ++i)
                if (first + i < n_mine) multiply(xv[from][i], wv[from][i], av[from][i]);
        };
        if (n_mine > 0) {
            if constexpr (with_w) fetch_a(0, 0);  // (the first loads of x and W are under way)
            else fetch(0, 0);
            for (int i = 0; i < n_mine; i += 2 * kAhead) {
                if (i + kAhead < n_mine) fetch(1, i + kAhead);
                use(0, i);
                if (i + 2 * kAhead < n_mine) fetch(0, i + 2 * kAhead);
                if (i + kAhead < n_mine) use(1, i + kAhead);
            }
        }
        if (whole * 16 < K && wave == whole % kOneWaves) {  // the turn that K ends in
            floatx4 wt{0.f, 0.f, 0.f, 0.f}, at_[kBlocks];
            const floatx4 xt = load4_until(xr, whole * 16, K - g * 4);
            if constexpr (with_w) wt = load4_until(wr, whole * 16, K - g * 4);
#pragma unroll
            for (int p = 0; p < blocks; ++p) at_[p] = load4_until(ar[p], whole * 16, K - g * 4);
            multiply(xt, wt, at_);
        }
        // the waves' sums meet in LDS and are added in wave order; a lane holds columns 4 g .. + 3 of row m
        if constexpr (with_w) *reinterpret_cast<floatx4 *>(&s_sum[wave][m][g * 4]) = acc[0] + acc[1];
#pragma unroll
        for (int p = 0; p < blocks; ++p) *reinterpret_cast<floatx4 *>(&s_sum[wave][m][kOneTile + p * 16 + g * 4]) = accv[p][0] + accv[p][1];
        __syncthreads();
        auto sum_of = [&](int row, int c) __attribute__((always_inline)) {
            float s = s_sum[0][row][c];
#pragma unroll
            for (int w = 1; w < kOneWaves; ++w) s += s_sum[w][row][c];
            return s;
        };
        if constexpr (with_w) sum = sum_of(rl, tid % kOneTile);
        if constexpr (blocks > 0) {
            for (int e = tid; e < kOneTile * 16 * blocks; e += 64 * kOneWaves) s_v[e / (16 * blocks)][e % (16 * blocks)] = sum_of(e / (16 * blocks), kOneTile + e % (16 * blocks));
            __syncthreads();
            // what these ranks give of the thread's B_i v
            if (my_slot >= 0) {
                const int end = min(my_rank, first_rank + kOneRanks - my_off);
                int j = max(first_rank - my_off, 0);
                const float *const v = &s_v[rl][0] + my_off - first_rank;
                if (j == 0) {
#pragma unroll
                    for (int q = 0; q < kEarly; ++q)
                        if (4 * q + 4 <= end) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) d = fmaf(v[4 * q + i], early[q][i], d);
                            j = 4 * q + 4;
                        }
                }
                for (; j < end; ++j) d = fmaf(v[j], Bn[j], d);
            }
        }
    };
    if (total == 0) walk(std::true_type{}, std::integral_constant<int, 0>{}, 0);
    else if (total <= 16) walk(std::true_type{}, std::integral_constant<int, 1>{}, 0);
    else walk(std::true_type{}, std::integral_constant<int, 2>{}, 0);
    for (int first_rank = kOneRanks; first_rank < total; first_rank += kOneRanks) {
        __syncthreads();  // (what the walk before left has been read)
        walk(std::false_type{}, std::integral_constant<int, 2>{}, first_rank);
    }
    if (t0 + rl < T && n < N) y[(size_t)(t0 + rl) * N + n] = my_slot >= 0 ? sum + my_scale * d : sum;
}

// Where the call's rows meet at most 32 ranks whichever adapters they name, so that one walk over K is enough (with a second
// one 8 rows 256 x 512 take 8.3 us, on two launches 7.4), K is short (16 rows of rank 8: 700 x 700 two launches 8.1 us / one
// 7.7, 1000 x 1000 9.1 / 10.4: the ranks are read by every workgroup) and two workgroups per compute unit are all there are.
// Adapters loaded later, under a captured graph, only add walks.  (A pool that holds none yet says nothing of the ranks to come: two
// launches.)  As the count of loaded adapters decides, a load can move the next call to the other form, which adds in another order.
// W and adapters read for the first time, two launches / one: 8 rows 512 x 512 10.5 / 8.9 us, 16 rows 700 x 700 12.5 / 9.2, 300 x 2000
// 10.4 / 7.7.
long long one_tiles(int T, int N) { return (((long long)T + kOneTile - 1) / kOneTile) * (((long long)N + kOneTile - 1) / kOneTile); }
// (n_segments: how many different adapters the routing tables can name)
bool one_launch(int T, int K, int N, int n_loaded, int max_rank, int n_segments)
{
    return n_loaded > 0 && (long long)std::min({kOneTile, T, n_loaded, n_segments}) * max_rank <= kOneRanks && K <= 700 && one_tiles(T, N) <= 512;
}

// A launch holds fewer than 2^32 threads: rows of the shrink, and tiles of the product, beyond that many workgroups go into
// further launches.
constexpr size_t kMaxGroups = ((size_t)1 << 32) / kThreads - 1;
size_t launches_of(size_t workgroups) { return (workgroups + kMaxGroups - 1) / kMaxGroups; }

// 16 x 16 outputs where such tiles leave a quarter of the compute units free (and for up to 16 rows), else 32 x 32, which loads half
// as much per product, unless 32 x 16 come out as one round of workgroups.  Two launches, 16 x 16 / 32 x 16 / 32 x 32: 60 rows
// 700 x 700 (176 tiles of 16) 8.7 / 10.5 / 12.2 us, 270 rows 300 x 400 (425) 8.1 / 8.4 / 9.8, 60 rows 2048 x 2048 (512; 256 of
// 32 x 16) 21.3 / 18.2 / 22.6, 155 rows 1000 x 1430 (900; 450) 19.8 / 19.3 / 17.0, 1430 x 1000 (630; 315) 22.0 / 24.3 / 18.2.
// (Between 193 and 511 tiles of 16 x 16 the two are within 4 % of each other; there a call keeps the 32 x 16 that it has always had.)
struct Tiles {
    int mb, nb;
    size_t n;
};
Tiles choose_tiles(int T, int N)
{
    const size_t m16 = ((size_t)T + 15) / 16, m32 = ((size_t)T + 31) / 32, n16 = ((size_t)N + 15) / 16, n32 = ((size_t)N + 31) / 32;
    if (T <= 16 || m16 * n16 <= 192) return {1, 1, m16 * n16};
    if (m32 * n16 <= 256) return {2, 1, m32 * n16};
    return {2, 2, m32 * n32};
}

}  // namespace

void elora::fp32_plan(const elora_linear_desc_t &d, elora_plan_t *plan)
{
    const int T = std::max(d.n_tokens, 1);
    const size_t tiles = choose_tiles(T, d.d_out).n;
    if (d.pool && one_launch(T, d.d_in, d.d_out, d.pool->n_loaded, d.pool->max_rank, d.adapter_idx ? T : d.n_segments)) {
        plan->n_launches = 1;
        plan->grid = (int)one_tiles(T, d.d_out);
        return;
    }
    plan->n_launches = (int)(launches_of(tiles) + (d.pool ? launches_of((size_t)T) : 0));
    plan->grid = (int)std::min(tiles, kMaxGroups);
}

int elora::launch_fp32(const LinearArgs &a, hipStream_t stream)
{
    int32_t *const row_slot = reinterpret_cast<int32_t *>(a.ws + a.wsl.row_slot);
    float *const row_scale = reinterpret_cast<float *>(a.ws + a.wsl.row_scale), *const V = reinterpret_cast<float *>(a.ws + a.wsl.v);
    const float *const x = static_cast<const float *>(a.x), *const W = static_cast<const float *>(a.W);
    const int R = a.pool.max_rank;
    if (a.has_pool && one_launch(a.T, a.K, a.N, a.n_loaded, R, a.route.adapter_idx ? a.T : a.route.n_segments)) {
        profile_mark_begin(stream);
        hipLaunchKernelGGL(fp32_one_kernel, dim3((unsigned)one_tiles(a.T, a.N)), dim3(64 * kOneWaves), 0, stream, a.T, a.K, a.N, x, W, a.pool, a.route, static_cast<float *>(a.y));
        ELORA_HIP_TRY(hipGetLastError());
        profile_mark_end(stream);
        return ELORA_OK;
    }
    for (size_t t = 0; a.has_pool && t < (size_t)a.T; t += kMaxGroups) {
        // (a wave per two rank entries, none that has nothing to do)
        hipLaunchKernelGGL(fp32_shrink_kernel, dim3((unsigned)std::min((size_t)a.T - t, kMaxGroups), (R + kPiece - 1) / kPiece), dim3(64 * std::min((R + 1) / 2, kWaves)), 0, stream, a.K, x, a.route,
                           a.pool, row_slot, row_scale, V, R, (int)t);
        ELORA_HIP_TRY(hipGetLastError());
    }
    const Tiles tiles = choose_tiles(a.T, a.N);
    auto go = [&](auto kern) -> int {
        for (size_t first = 0; first < tiles.n; first += kMaxGroups) {
            hipLaunchKernelGGL(kern, dim3((unsigned)std::min(tiles.n - first, kMaxGroups)), dim3(kThreads), 0, stream, a.T, a.K, a.N, x, W, a.pool,
                               a.has_pool ? 1 : 0, row_slot, row_scale, V, R, static_cast<float *>(a.y), (int)first);
            ELORA_HIP_TRY(hipGetLastError());
        }
        return ELORA_OK;
    };
    profile_mark_begin(stream);
    const int rc = tiles.mb == 1 ? go(fp32_product_kernel<1, 1, 1>) : tiles.nb == 1 ? go(fp32_product_kernel<2, 1, 2>) : go(fp32_product_kernel<2, 2, 1>);
    if (rc == ELORA_OK) profile_mark_end(stream);
    return rc;
}
