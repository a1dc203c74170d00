// One word of the group product a [x] b (paper section 2.2) of two flat elements in memory, for the kernels that form
// products of rows of signatures.
#ifndef SIG_PRODUCT_H_
#define SIG_PRODUCT_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sig {

// The cross terms of the word at flat position p, TERMS = its length less one, added to acc one after the other from
// the longest prefix to the shortest.  No level table is read: the word without its last letter sits at p / d - 1 (level
// k + 1 starts at d times the start of level k, plus d), and level m + 1 of the suffixes at d off_m + d.  The letters are
// peeled off before anything is loaded, so that every load of the word is in flight together; a word costs one trip to
// memory where a loop that adds as it loads takes one per term.
// V is T, or several consecutive words that differ in their last letter only: they share their scalars of `a` and their
// letters, and lie side by side in `b` and in the result.
template <int TERMS, typename T, typename V>
__device__ __forceinline__ V product_cross_terms(const T *a, const T *b, uint32_t p, uint32_t d, V acc)
{
    T x[TERMS];
    V y[TERMS];
    uint32_t suffix = 0, scale = 1, off = 0;
#pragma unroll
    for (int t = 0; t < TERMS; ++t) {
        const uint32_t q = p / d;
        suffix += (p - q * d) * scale;
        p = q - 1;
        x[t] = a[p];
        y[t] = *reinterpret_cast<const V *>(b + off + suffix);
        scale *= d;
        off = off * d + d;
    }
#pragma unroll
    for (int t = 0; t < TERMS; ++t) acc += x[t] * y[t];
    return acc;
}

// The word (words) at position p < S < 2^31 of a [x] b; D > 0: the channel count as a constant.
template <typename T, typename V, int D>
__device__ __forceinline__ V product_word(const T *a, const T *b, uint32_t p, uint32_t d_runtime)
{
    const uint32_t d = D > 0 ? uint32_t(D) : d_runtime;
    int k = 1;
    for (uint32_t size = d, end = d; p >= end; ++k) {
        size *= d;
        end += size;
    }
    V acc = *reinterpret_cast<const V *>(a + p) + *reinterpret_cast<const V *>(b + p);
    switch (k) {
        case 1: return acc;
        case 2: return product_cross_terms<1, T, V>(a, b, p, d, acc);
        case 3: return product_cross_terms<2, T, V>(a, b, p, d, acc);
        case 4: return product_cross_terms<3, T, V>(a, b, p, d, acc);
        case 5: return product_cross_terms<4, T, V>(a, b, p, d, acc);
        case 6: return product_cross_terms<5, T, V>(a, b, p, d, acc);
        case 7: return product_cross_terms<6, T, V>(a, b, p, d, acc);
        case 8: return product_cross_terms<7, T, V>(a, b, p, d, acc);
        case 9: return product_cross_terms<8, T, V>(a, b, p, d, acc);
    }
    uint32_t suffix = 0, scale = 1, off = 0;
    for (int t = 1; t < k; ++t) {
        const uint32_t q = p / d;
        suffix += (p - q * d) * scale;
        p = q - 1;
        acc += a[p] * *reinterpret_cast<const V *>(b + off + suffix);
        scale *= d;
        off = off * d + d;
    }
    return acc;
}

// Four consecutive words as a vector, where the channel count is divisible by four and the rows are aligned to four scalars.
template <typename T>
struct Four {
    typedef T type __attribute__((ext_vector_type(4)));
};

// All the words of one prefix, W = d of them, with the alignment of a scalar.
template <typename T, int W>
struct Siblings {
    T v[W];
    __device__ __forceinline__ Siblings operator+(const Siblings &o) const
    {
        Siblings r;
#pragma unroll
        for (int i = 0; i < W; ++i) r.v[i] = v[i] + o.v[i];
        return r;
    }
    __device__ __forceinline__ void operator+=(const Siblings &o)
    {
#pragma unroll
        for (int i = 0; i < W; ++i) v[i] += o.v[i];
    }
    friend __device__ __forceinline__ Siblings operator*(T x, const Siblings &y)
    {
        Siblings r;
#pragma unroll
        for (int i = 0; i < W; ++i) r.v[i] = x * y.v[i];
        return r;
    }
};

}  // namespace sig

#endif  // SIG_PRODUCT_H_
