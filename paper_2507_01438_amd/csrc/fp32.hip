// The fp32 path (any shape, any rank): two launches.
//   route + shrink   per row: pool slot and scale (Sec. 3.4: each request names its adapter), v_t = A_i x_t
//   product          y_t = W x_t + s * B_i v_t, written at row t (Sec. 3.4 closing equation)
// Calls of this path are small (a model kept in fp32 to check an adapter), so what bounds them is latency: few launches, every
// load of a wave under way at once, and K split over the waves of a workgroup so that a call of a few rows still has a
// wave on most compute units.  Products and sums are fp32 throughout, on the fp32 matrix instructions.  Calls with rank-16
// adapters, three launches of plain FMAs through 64 x 64 tiles / here: 8 rows 512 x 512 67 / 9.5 us, 155 rows 1000 x 1430
// 162 / 21, 272 rows 2048 x 3000 317 / 81, 2000 rows 2048 x 2048 615 / 294, 4096 rows 4096 x 4096 4182 / 2198 (there the
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
// A launch with at most two workgroups per compute unit has four turns' loads of a wave under way; with more of them it is the
// other workgroups that hide a load, and with one turn ahead four of them fit (the 32 x 32 tile with four ahead: 157 registers,
// one workgroup): rank-8 calls, four ahead / one, 272 rows 1000 x 3000 50 / 42 us, 2000 rows 128 x 10000 440 / 144, 2048 x 10000
// 1556 / 1336; 256 rows 2048 x 2048 45 / 40.
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

// A launch holds fewer than 2^32 threads: rows of the shrink, and tiles of the product, beyond that many workgroups go into
// further launches.
constexpr size_t kMaxGroups = ((size_t)1 << 32) / kThreads - 1;
size_t launches_of(size_t workgroups) { return (workgroups + kMaxGroups - 1) / kMaxGroups; }

// The largest tile that still gives every compute unit a workgroup: a turn of 32 x 32 outputs loads half as much per product
// as one of 32 x 16.
struct Tiles {
    int mb, nb;
    size_t n;
};
Tiles choose_tiles(int T, int N)
{
    const size_t m32 = ((size_t)T + 31) / 32, n16 = ((size_t)N + 15) / 16, n32 = ((size_t)N + 31) / 32;
    if (T <= 16) return {1, 1, n16};
    if (m32 * n32 < 256) return {2, 1, m32 * n16};
    return {2, 2, m32 * n32};
}

}  // namespace

void elora::fp32_plan(const elora_linear_desc_t &d, elora_plan_t *plan)
{
    const int T = std::max(d.n_tokens, 1);
    const size_t tiles = choose_tiles(T, d.d_out).n;
    plan->n_launches = (int)(launches_of(tiles) + (d.pool ? launches_of((size_t)T) : 0));
    plan->grid = (int)std::min(tiles, kMaxGroups);
}

int elora::launch_fp32(const LinearArgs &a, hipStream_t stream)
{
    int32_t *const row_slot = reinterpret_cast<int32_t *>(a.ws + a.wsl.row_slot);
    float *const row_scale = reinterpret_cast<float *>(a.ws + a.wsl.row_scale), *const V = reinterpret_cast<float *>(a.ws + a.wsl.v);
    const float *const x = static_cast<const float *>(a.x), *const W = static_cast<const float *>(a.W);
    const int R = a.pool.max_rank;
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
    const int rc = tiles.mb == 1 ? (tiles.n > 512 ? go(fp32_product_kernel<1, 1, 1>) : go(fp32_product_kernel<1, 1, 4>))
                   : tiles.nb == 1 ? go(fp32_product_kernel<2, 1, 4>) : go(fp32_product_kernel<2, 2, 1>);
    if (rc == ELORA_OK) profile_mark_end(stream);
    return rc;
}
