// What the kernels that take sixteen increments at a time share: sums over the sixteen lanes of a row, and products of 32-bit numbers on
// the matrix cores' bfloat16 instructions.
//
// Operands are 32-bit numbers cut into three bfloat16 pieces of 8 bits, high, middle and low (exact: each piece is the truncated rest
// of the one before), of whose nine products the six to eight largest are summed in fp32, the small ones first; what is left
// out is 2^-24 of a term and less.  A sum of 16 such terms is off by 7.7e-8 of its norm where a chain of fp32 multiply-adds is off by 7.4e-8.
// The matrix cores take them at 16 times the fp32 rate, so six products are 2.7 times as fast as one fp32 instruction.
// An infinity has no such pieces (its rest is not a number, nor is infinity times a zero piece): where a result would be infinite, by overflow or because a
// point or a cotangent is, these kernels give NaN.  Which results are finite is the same as on the other kernels.
#ifndef SIG_TILE_COMMON_H_
#define SIG_TILE_COMMON_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sig_lane_ops.h"

namespace sig {
namespace {

typedef __bf16 TlHalves __attribute__((ext_vector_type(8)));
typedef unsigned TlWords __attribute__((ext_vector_type(4)));

__host__ __device__ constexpr int64_t tl_pow(int d, int k)
{
    int64_t p = 1;
    for (int i = 0; i < k; ++i) p *= d;
    return p;
}

__host__ __device__ constexpr int64_t tl_off(int d, int k)   // offset of level k (1-based) in a flat element
{
    int64_t off = 0;
    for (int j = 1; j < k; ++j) off += tl_pow(d, j);
    return off;
}

__host__ __device__ constexpr float tl_inv_factorial(int n)
{
    double f = 1;
    for (int i = 2; i <= n; ++i) f *= i;
    return float(1 / f);
}

__device__ __forceinline__ unsigned tl_bits(float x) { return __builtin_bit_cast(unsigned, x); }
__device__ __forceinline__ float tl_float(unsigned x) { return __builtin_bit_cast(float, x); }

// The pieces of x, each in the upper half of a word.
struct TlPieces {
    unsigned h, m, l;
};
__device__ __forceinline__ TlPieces tl_split(float x)
{
    TlPieces p;
    p.h = tl_bits(x) & 0xffff0000u;
    const float r = x - tl_float(p.h);
    p.m = tl_bits(r) & 0xffff0000u;
    p.l = tl_bits(r - tl_float(p.m));
    return p;
}
__device__ __forceinline__ unsigned tl_pack(unsigned first, unsigned second) { return __builtin_amdgcn_perm(second, first, 0x07060302u); }

__device__ __forceinline__ f4 tl_mfma(TlWords a, TlWords b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(TlHalves, a), __builtin_bit_cast(TlHalves, b), c, 0, 0, 0);
}

// Over the sixteen lanes of a row: the value SHIFT lanes up or down (zero beyond the row), lane 0's and lane 15's.
template <int SHIFT>
__device__ __forceinline__ float tl_up(float v)
{
    return tl_float(__builtin_amdgcn_update_dpp(0, int(tl_bits(v)), 0x100 + SHIFT, 0xf, 0xf, true));
}
template <int SHIFT>
__device__ __forceinline__ float tl_down(float v)
{
    return tl_float(__builtin_amdgcn_update_dpp(0, int(tl_bits(v)), 0x110 + SHIFT, 0xf, 0xf, true));
}
__device__ __forceinline__ float tl_first(float v)
{
    return tl_float(__builtin_amdgcn_update_dpp(0, int(tl_bits(v)), 0x150, 0xf, 0xf, true));   // row_newbcast:0
}
__device__ __forceinline__ float tl_last(float v)
{
    return tl_float(__builtin_amdgcn_update_dpp(0, int(tl_bits(v)), 0x15f, 0xf, 0xf, true));
}

// Sums from the lane to the end of the row, and from its start to the lane, of several values step by step side by side: a step waits two
// instructions for the one before.
template <int COUNT>
__device__ __forceinline__ void tl_suffixes(float (&v)[COUNT])
{
    const auto step = [&](auto shift) {
#pragma unroll
        for (int i = 0; i < COUNT; ++i) v[i] += tl_up<decltype(shift)::value>(v[i]);
        if (COUNT > 1) __builtin_amdgcn_sched_barrier(0);
    };
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 8>{});
}
template <int COUNT>
__device__ __forceinline__ void tl_prefixes(float (&v)[COUNT])
{
    const auto step = [&](auto shift) {
#pragma unroll
        for (int i = 0; i < COUNT; ++i) v[i] += tl_down<decltype(shift)::value>(v[i]);
        if (COUNT > 1) __builtin_amdgcn_sched_barrier(0);
    };
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 8>{});
}
__device__ __forceinline__ float tl_suffix(float v)
{
    float x[1] = {v};
    tl_suffixes(x);
    return x[0];
}
__device__ __forceinline__ float tl_prefix(float v)
{
    float x[1] = {v};
    tl_prefixes(x);
    return x[0];
}

// In rows 0 and 2 the sum of a over the pair of rows, in rows 1 and 3 that of b.
__device__ __forceinline__ float tl_rows_16(float a, float b)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane16_swap(tl_bits(a), tl_bits(b), false, false);
    const unsigned x = r[0], y = r[1];
    return tl_float(x) + tl_float(y);
}
// In rows 0 and 1 the sum of a over the two halves of the wavefront, in rows 2 and 3 that of b.
__device__ __forceinline__ float tl_rows_32(float a, float b)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 r = __builtin_amdgcn_permlane32_swap(tl_bits(a), tl_bits(b), false, false);
    const unsigned x = r[0], y = r[1];
    return tl_float(x) + tl_float(y);
}

// Orders a wavefront's own LDS writes before its reads of what other lanes wrote.
__device__ __forceinline__ void tl_wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

}  // namespace
}  // namespace sig

#endif  // SIG_TILE_COMMON_H_
