// What the kernels that take sixteen increments at a time share: sums over the sixteen lanes of a row, and products of 32-bit numbers on
// the matrix cores' bfloat16 instructions.
//
// Operands are 32-bit numbers cut into three bfloat16 pieces of 8 bits, high, middle and low (exact: each piece is what is left of those before),
// of whose nine products six or eight are summed in fp32, the small ones first (the known way to products of 32-bit numbers on units for 16).  The matrix cores take them at 16 times the fp32 rate, so six products
// are 2.7 times as fast as one fp32 instruction.  Truncated, a middle piece is below 2^-7 of its number and a low one below 2^-15, of its sign.
//  - Eight products (gradients up to eight channels) leave out the low pieces' one, 2^-30 of a term.
//  - Six leave out up to 2^-21 of a term and 2^-23 in the mean, of the term's sign, where a multiply-add rounds off 2^-24.  The scan has a rounding per tile
//    instead of one per increment, and is 0.77 to 0.9 as far off as the prefix tree all the same; rounded pieces, 3 to 5 % of its time, brought 0.73 to 0.84.
//  - Gradients from nine channels on take six too, but the pieces of the increments are rounded to nearest, at most 2^-8 and 2^-17 and of either sign:
//    1.5 2^-23 of a term is left out, and does not add up over terms.
// An infinity has no such pieces (its rest is not a number, nor is infinity times a zero piece), and a product of two increments may overflow where the
// scalar that it is a factor of would not.  A signature with a scalar that is not finite is therefore formed once more, one increment after the other
// (tl_one_by_one).  A gradient that would be infinite, because a cotangent is or by overflow, comes out as NaN.
#ifndef SIG_TILE_COMMON_H_
#define SIG_TILE_COMMON_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sig_internal.h"
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

// The pieces of x, each in the upper half of a word: every piece what is left of those before, truncated.
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
// The upper or the lower halves of two words, the first's in the lower half.
__device__ __forceinline__ unsigned tl_pack(unsigned first, unsigned second) { return __builtin_amdgcn_perm(second, first, 0x07060302u); }
__device__ __forceinline__ unsigned tl_pack_lower(unsigned first, unsigned second) { return __builtin_amdgcn_perm(second, first, 0x05040100u); }
// The pieces of two numbers, packed: truncated,
__device__ __forceinline__ TlPieces tl_split_pair(float a, float b)
{
    const TlPieces p = tl_split(a), q = tl_split(b);
    return {tl_pack(p.h, q.h), tl_pack(p.m, q.m), tl_pack(p.l, q.l)};
}
// or rounded to nearest.  (Above the largest bfloat16 the nearest is an infinity: the high piece of such a number is that largest.)
__device__ __forceinline__ unsigned tl_nearest(float a, float b)
{
    typedef float F2 __attribute__((ext_vector_type(2)));
    typedef __bf16 B2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector((F2{a, b}), B2));
}
__device__ __forceinline__ TlPieces tl_split_pair_nearest(float a, float b)
{
    constexpr float most = 3.38953139e38f;   // 2^128 - 2^120
    const unsigned h = tl_nearest(__builtin_amdgcn_fmed3f(a, -most, most), __builtin_amdgcn_fmed3f(b, -most, most));
    const float ra = a - tl_float(h << 16), rb = b - tl_float(h & 0xffff0000u);
    const unsigned m = tl_nearest(ra, rb);
    return {h, m, tl_nearest(ra - tl_float(m << 16), rb - tl_float(m & 0xffff0000u))};
}

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

// One increment after the other, for paths whose scalars overflow or are no numbers: the word u of N - 1 letters, its prefixes and its children,
// formed as in sig_tree_impl.h.  visit(s, a, leaf) behind increment s: a[k] is the prefix of k letters, leaf the children.  The increments end at the
// n_inc points from `at` on, the first starts from `base` (null: the origin); the signature from `initial` (null: the identity).
template <int D, int N, typename Visit>
__device__ __forceinline__ void tl_one_by_one(const float *at, int64_t n_inc, const float *base, const float *initial, int u, Visit visit)
{
    constexpr int P = N - 1;
    int letter[P + 1];
    float a[P + 1], leaf[D], lo[D];
    int rest = u;
#pragma unroll
    for (int k = P; k >= 1; --k) {
        letter[k] = rest % D;
        a[k] = initial != nullptr ? initial[tl_off(D, k) + rest] : 0.f;
        rest /= D;
    }
#pragma unroll
    for (int c = 0; c < D; ++c) {
        leaf[c] = initial != nullptr ? initial[tl_off(D, N) + int64_t(u) * D + c] : 0.f;
        lo[c] = base != nullptr ? base[c] : 0.f;
    }
#pragma unroll 1
    for (int64_t s = 0; s < n_inc; ++s, at += D) {
        float z[D], h[N + 1];
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const float hi = at[c];
            z[c] = hi - lo[c];
            lo[c] = hi;
        }
#pragma unroll
        for (int i = 1; i <= P; ++i) {
            float zi = z[0];
#pragma unroll
            for (int c = 1; c < D; ++c) zi = letter[i] == c ? z[c] : zi;
            const float before = a[i];
            a[i] = i == 1 ? before + zi : __builtin_fmaf(h[i], zi, before);
#pragma unroll
            for (int k = i + 1; k <= N; ++k) {
                const float r = 1.f / float(k - i + 1);
                h[k] = i == 1 ? __builtin_fmaf(zi, r, before) : __builtin_fmaf(h[k], zi * r, before);
            }
        }
#pragma unroll
        for (int c = 0; c < D; ++c) leaf[c] = __builtin_fmaf(h[N], z[c], leaf[c]);
        visit(s, a, leaf);
    }
}

// That word, its children and the prefixes it is the first below into a signature.
template <int D, int N>
__device__ __forceinline__ void tl_store_word(float *out, int u, const float (&a)[N], const float (&leaf)[D])
{
#pragma unroll
    for (int c = 0; c < D; ++c) out[tl_off(D, N) + int64_t(u) * D + c] = leaf[c];
#pragma unroll
    for (int k = N - 1; k >= 1; --k) {
        const int below = int(tl_pow(D, N - 1 - k));
        if (u % below == 0) out[tl_off(D, k) + u / below] = a[k];
    }
}

}  // namespace
}  // namespace sig

#endif  // SIG_TILE_COMMON_H_
