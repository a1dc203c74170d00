// What a thread of the prefix-tree kernels does with the signature C of a neighbouring stretch of its path, with no help from
// other threads.  A thread stands for a word u = u_1 .. u_P and holds the scalars of its prefixes and of some levels below it.
//   * The signature A of what came before times C needs, at a word w, A at the prefixes of w and C at its suffixes:
//     (A [x] C)[w] = A[w] + C[w] + sum_j A[w_1 .. w_j] C[w_{j+1} ..].  The prefixes of the thread's words are its own.
//   * The gradient g with respect to a product S [x] C, carried back to S, is g'[w] = g[w] + sum_v g[w v] C[v] (|v| >= 1).  It is
//     linear in g, so where the gradient of a prefix is kept split over the threads below it, each carries its part by itself.
// Either reads C at the words made of the thread's last letters (and what is below them): some dozen scalars next to each other
// per level, which the lanes of a path read from the same few lines.
#ifndef SIG_STRETCH_OPS_H_
#define SIG_STRETCH_OPS_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sig {

__host__ __device__ constexpr int64_t stretch_off(int d, int k)   // offset of level k (1-based) in a flat element
{
    int64_t off = 0, p = 1;
    for (int j = 1; j < k; ++j) {
        p *= d;
        off += p;
    }
    return off;
}

// Scalar offset in a flat element of the word u_{j+1} .. u_i (1 <= i - j), and of the words below it.
template <int D>
__device__ __forceinline__ uint32_t suffix_word(const uint32_t *pre, int j, int i)
{
    uint32_t w = pre[i], width = 1;
    for (int k = j; k < i; ++k) width *= D;
    return j > 0 ? w - pre[j] * width : w;
}

// The scalars of a flat element of less than 4 GB from i on: a wavefront's C is the same, so an address takes a lane one register.
template <typename T>
__device__ __forceinline__ const T *stretch_at(const T *C, uint32_t i)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(C) + i * uint32_t(sizeof(T)));
}

// What a thread reads of C for a product with it on the right.  Read and used apart, so that all reads of a product (and of the
// next one, see sig_stretch_group_kernel) are on their way together.  lo[i] is the scalar of the word's prefix of i letters, h1
// those of the words one letter longer than u; pre[i]: number of that prefix among the words of i letters.
template <typename T, int D, int P>
struct StretchFactor {
    T own[P + 1], cross[P + 1][P + 1], below[P + 1][D];

    __device__ __forceinline__ void read(const uint32_t *pre, const T *C)
    {
#pragma unroll
        for (int i = 1; i <= P; ++i) {
            own[i] = stretch_at(C, pre[i])[stretch_off(D, i)];
#pragma unroll
            for (int j = 1; j < i; ++j) cross[i][j] = stretch_at(C, suffix_word<D>(pre, j, i))[stretch_off(D, i - j)];
        }
#pragma unroll
        for (int j = 0; j <= P; ++j) {
            const T *r = j < P ? stretch_at(C, suffix_word<D>(pre, j, P) * D) + stretch_off(D, P - j + 1) : C;
#pragma unroll
            for (int c = 0; c < D; ++c) below[j][c] = r[c];
        }
    }
    // (lo, h1) <- (lo, h1) [x] C
    __device__ __forceinline__ void multiply(T *lo, T *h1) const
    {
#pragma unroll
        for (int c = 0; c < D; ++c) {
            T add = below[0][c];
#pragma unroll
            for (int j = 1; j <= P; ++j) add += lo[j] * below[j][c];
            h1[c] += add;
        }
#pragma unroll
        for (int i = P; i >= 1; --i) {
            T add = own[i];
#pragma unroll
            for (int j = 1; j < i; ++j) add += lo[j] * cross[i][j];
            lo[i] += add;
        }
    }
};

// The gradient (lo, h1, h2) of the thread's words and their prefixes carried back through a multiplication by C; h2, the top
// level, stays as it is.
template <typename T, int D, int P>
__device__ __forceinline__ void stretch_carry_back(T *lo, T *h1, const T *h2, const uint32_t *pre, const T *C)
{
#pragma unroll
    for (int i = 1; i <= P; ++i) {   // from what the longer words hold before they change themselves
        T cross[P + 1], r1[D], r2[D * D];
        const uint32_t rest = i < P ? suffix_word<D>(pre, i, P) : 0;   // the letters behind the prefix
#pragma unroll
        for (int j = i + 1; j <= P; ++j) cross[j] = stretch_at(C, suffix_word<D>(pre, i, j))[stretch_off(D, j - i)];
#pragma unroll
        for (int c = 0; c < D; ++c) r1[c] = stretch_at(C, rest * D)[stretch_off(D, P - i + 1) + c];
#pragma unroll
        for (int c = 0; c < D * D; ++c) r2[c] = stretch_at(C, rest * (D * D))[stretch_off(D, P - i + 2) + c];
        // every read is issued before the first is used, while they fit the registers beside the thread's own scalars
        if constexpr (D * int(sizeof(T)) <= 28) __builtin_amdgcn_sched_barrier(0);
        T sum[D];   // one running sum per last letter
#pragma unroll
        for (int e = 0; e < D; ++e) sum[e] = h1[e] * r1[e];
#pragma unroll
        for (int c = 0; c < D; ++c)
#pragma unroll
            for (int e = 0; e < D; ++e) sum[e] += h2[c * D + e] * r2[c * D + e];
#pragma unroll
        for (int j = i + 1; j <= P; ++j) sum[j % D] += lo[j] * cross[j];
        T add = sum[0];
#pragma unroll
        for (int e = 1; e < D; ++e) add += sum[e];
        lo[i] += add;
        if (i == P) {   // r1 is level 1 of C
#pragma unroll
            for (int c = 0; c < D; ++c) {
                T under = T(0);
#pragma unroll
                for (int e = 0; e < D; ++e) under += h2[c * D + e] * r1[e];
                h1[c] += under;
            }
        }
    }
}

}  // namespace sig

#endif  // SIG_STRETCH_OPS_H_
