// What the kernels of the GEMM path (route, shrink, matrix products) share.
#pragma once

#include <type_traits>

#include "common.h"

namespace elora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));

template <int V> using ic = std::integral_constant<int, V>;

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(ic<I>{});
        static_for<I + 1, N>(f);
    }
}

typedef __attribute__((address_space(3))) void *lptr_t;
// one direct load of the wave: 16 (4) bytes per lane from base + off to lds + 16 (4) * lane.  M0 holds the LDS address and
// needs a cycle to settle; nothing else of the kernels that use these keeps a value in M0 across statements.
__device__ __forceinline__ void dma16(uint32_t lds, const void *base, uint32_t off)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory");
}
__device__ __forceinline__ void dma4(uint32_t lds, const void *base, uint32_t off)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory");
}
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

constexpr int kXcds = 8;     // workgroup b runs on XCD b % 8
constexpr int kRankPad = 64; // rows of V (the shrink results) are padded to this many rank entries, with zeros

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }

// two floats -> packed bf16 pair, round-to-nearest-even (one v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    bf16x2_t v = __builtin_convertvector(float2_t{lo, hi}, bf16x2_t);
    return __builtin_bit_cast(uint32_t, v);
}

// A float as the sum of three bf16, exactly (down to 2^-133): the eight leading bits of its 24, the next eight and the last
// eight, cut off and not rounded, so that a part is finite where the float is.  Times an infinity the parts have to add up
// to what the float gives: all three have its sign, and none is zero unless the float is (a part that would be leaves the
// last unit of the one before it to it); of an infinity or a NaN every part is one.
__device__ __forceinline__ void split_bf16(float v, uint16_t part[3])
{
    const uint32_t u = __float_as_uint(v);
    if ((u & 0x7f800000u) == 0x7f800000u) {
        part[0] = part[1] = part[2] = (uint16_t)((u >> 16) | ((u & 0x007fffffu) != 0 ? 0x40u : 0u));
        return;
    }
    auto cut = [](uint32_t bits) { return (bits & 0xffffu) != 0 || bits << 1 == 0 ? bits >> 16 : (bits >> 16) - 1; };
    const uint32_t p0 = cut(u);
    const float r1 = v - __uint_as_float(p0 << 16);
    const uint32_t p1 = cut(__float_as_uint(r1));
    part[0] = (uint16_t)p0;
    part[1] = (uint16_t)p1;
    part[2] = (uint16_t)(__float_as_uint(r1 - __uint_as_float(p1 << 16)) >> 16);
}

// Eight consecutive values of an adapter kept in 8-bit blocks (they lie in one block: ranks and d_in are multiples of
// 8 there) as matrix-core operands: scale * code, exact in fp32, rounded once to bf16.  (The decode and generic
// kernels multiply the exact products; here the adapter passes through the matrix cores like every other operand.)
__device__ __forceinline__ u32x4 q8_to_bf16x8(u32x2 codes, float sc)
{
    u32x4 o;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const uint32_t w = codes[b >> 1] >> (16 * (b & 1));
        o[b] = pack_bf16x2(sc * (float)(int8_t)(w & 0xffu), sc * (float)(int8_t)((w >> 8) & 0xffu));
    }
    return o;
}

// The projections a shrink launch serves: one, or two or three that read the same x (q / k / v, gate / up), each with
// a pool and a workspace of its own.
constexpr int kShrinkMulti = 3;
struct ShrinkProj {
    PoolView pool;
    int32_t *row_slot;   // [T] from the route kernel
    float *row_scale;    // [T]
    int32_t *short_rows; // [T]: the rows that sit in runs shorter than kShortRun, in any order
    uint16_t *V;         // [T][Rpad] bf16(s * A_i x_t), zeros beyond the rank and in rows without adapter
    // Where the product takes the shrink results whole (band_whole): [2][T][Rpad] the second and third bf16 of A_i x_t, of
    // which V then holds the first (see split_bf16; the scale comes after the expand, as in the decode kernel).  Else nullptr.
    uint16_t *V_rest;
    float *part;         // fp32 sums of the K-slices: [tile][slice][kShrinkRows][Rpad]
    int *sync;           // the workspace's counters
    int Rpad;
};
struct ShrinkArgs {
    int n;               // projections
    int T, K;
    int n_tiles;         // kShrinkRows-row tiles
    int ks;              // K-slices per tile
    int wgs_per_xcd;     // workgroups per projection and XCD
    bool by_row;         // rings as for ranks up to 32: most rows sit in short runs
    bool rows_apart;     // the rows of short runs are a launch of their own
    const uint16_t *x;
    ShrinkProj proj[kShrinkMulti];
};

// everything the launches below need; whole[i]: projection i's product takes the shrink results whole
void shrink_args(ShrinkArgs &s, const LinearArgs *a, int n, const bool *whole);
int launch_route(const ShrinkArgs &s, const LinearArgs *a, bool copy, hipStream_t stream);  // copy: and the bf16 copy of a[0]'s 4-bit or 8-bit W into a[0].wsl.wdeq
int launch_shrink(const ShrinkArgs &s, hipStream_t stream);

}  // namespace elora
