// Group product of two batches of truncated signatures, out[b] = a[b] [x] b[b]
// (paper section 2.2:  (A [x] B)_k = sum_{j=0..k} A_j (x) B_{k-j},  A_0 = B_0 = 1; by Chen's
// identity, eq. "grouplike", this joins the signatures of two adjacent intervals, section 5.5).
//
// One thread per output word w = w_1..w_k:
//     out_k[w] = a_k[w] + b_k[w] + sum_{j=1..k-1} a_j[w_1..w_j] * b_{k-j}[w_{j+1}..w_k].
// Consecutive threads share the prefix (one broadcast read of a) and walk consecutive suffixes
// (coalesced reads of b), so the kernel runs at memory speed: 3 S scalars per path.
#include "sig_internal.h"
#include "sig_product.h"

namespace sig {
namespace {

// Where product p finds its operands: with p = q * n_inner + i (i < n_inner), operand a starts at
// a + q * a_outer + i * a_inner scalars, likewise b and out.  Packed operands: n_inner = everything, inner = S.
struct Strides {
    int64_t a, b, out;                    // inner strides
    int64_t n_inner;                      // products per outer step
    int64_t a_outer, b_outer, out_outer;  // outer strides
};

// D: the channel count when it is one of the common ones (division by a constant is a multiply and a shift), 0 for any
// other d (division by the runtime value).
// V = several consecutive words per thread that differ only in their last letter: each term is one broadcast scalar of `a`
// times consecutive scalars of `b`, and the letters are worked out once for all of them.  Four words, moved as vectors, for
// channel counts that are multiples of 4 (then every level size and offset is a multiple of 4 too), else all d words of a
// prefix: 0.6 the time of a word per thread at d = 5 and 7 (tree of products, 128 paths).
template <typename T, typename V, int D>
__global__ void __launch_bounds__(256)
sig_combine_kernel(Shape sh, Strides rs, const T *__restrict__ a, const T *__restrict__ b, T *__restrict__ out)
{
    constexpr uint32_t kWords = sizeof(V) / sizeof(T);
    static_assert(kWords == 1 || D % kWords == 0, "the words of a thread share their prefix");
    const uint32_t n = uint32_t(sh.S) / kWords;
    for (int64_t p = blockIdx.y; p < sh.B; p += gridDim.y) {
        const int64_t q = p / rs.n_inner, r = p - q * rs.n_inner;
        const T *ap = a + q * rs.a_outer + r * rs.a;
        const T *bp = b + q * rs.b_outer + r * rs.b;
        T *op = out + q * rs.out_outer + r * rs.out;
        for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
            *reinterpret_cast<V *>(op + kWords * v) = product_word<T, V, D>(ap, bp, kWords * v, uint32_t(sh.d));
    }
}

template <typename T>
hipError_t launch_combine(const Shape &sh, const T *a, const T *b, T *out, hipStream_t st, const int64_t *strides)
{
    // strides: {a, b, out} or {a, b, out, n_inner, a_outer, b_outer, out_outer} (flagged by a negative first entry
    // being impossible: the caller passes the count in strides[3] as 0 when there is no outer level)
    const int64_t whole = int64_t(1) << 62;
    Strides rs = {sh.S, sh.S, sh.S, whole, 0, 0, 0};
    if (strides != nullptr) {
        rs.a = strides[0];
        rs.b = strides[1];
        rs.out = strides[2];
        if (strides[3] > 0) {
            rs.n_inner = strides[3];
            rs.a_outer = strides[4];
            rs.b_outer = strides[5];
            rs.out_outer = strides[6];
        }
    }
    const unsigned bx = unsigned((sh.S + 255) / 256 < 4096 ? (sh.S + 255) / 256 : 4096);
    const unsigned by = unsigned(sh.B < 65535 ? sh.B : 65535);
    const dim3 grid(bx, by), block(256);
    const bool aligned = (reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(out)) %
                                 (4 * sizeof(T)) == 0 &&
                         (rs.a | rs.b | rs.out | rs.a_outer | rs.b_outer | rs.out_outer) % 4 == 0;
    typedef typename Four<T>::type V4;
    if (aligned && (sh.d == 4 || sh.d == 8 || sh.d == 16)) {
        const dim3 grid4(unsigned((sh.S / 4 + 255) / 256 < 4096 ? (sh.S / 4 + 255) / 256 : 4096), by);
        if (sh.d == 4) hipLaunchKernelGGL((sig_combine_kernel<T, V4, 4>), grid4, block, 0, st, sh, rs, a, b, out);
        if (sh.d == 8) hipLaunchKernelGGL((sig_combine_kernel<T, V4, 8>), grid4, block, 0, st, sh, rs, a, b, out);
        if (sh.d == 16) hipLaunchKernelGGL((sig_combine_kernel<T, V4, 16>), grid4, block, 0, st, sh, rs, a, b, out);
        return hipGetLastError();
    }
    const dim3 grid_d(unsigned((sh.S / sh.d + 255) / 256 < 4096 ? (sh.S / sh.d + 255) / 256 : 4096), by);
    switch (sh.d) {
        case 2: hipLaunchKernelGGL((sig_combine_kernel<T, Siblings<T, 2>, 2>), grid_d, block, 0, st, sh, rs, a, b, out); break;
        case 3: hipLaunchKernelGGL((sig_combine_kernel<T, Siblings<T, 3>, 3>), grid_d, block, 0, st, sh, rs, a, b, out); break;
        case 4: hipLaunchKernelGGL((sig_combine_kernel<T, T, 4>), grid, block, 0, st, sh, rs, a, b, out); break;
        case 5: hipLaunchKernelGGL((sig_combine_kernel<T, Siblings<T, 5>, 5>), grid_d, block, 0, st, sh, rs, a, b, out); break;
        case 6: hipLaunchKernelGGL((sig_combine_kernel<T, Siblings<T, 6>, 6>), grid_d, block, 0, st, sh, rs, a, b, out); break;
        case 7: hipLaunchKernelGGL((sig_combine_kernel<T, Siblings<T, 7>, 7>), grid_d, block, 0, st, sh, rs, a, b, out); break;
        case 8: hipLaunchKernelGGL((sig_combine_kernel<T, T, 8>), grid, block, 0, st, sh, rs, a, b, out); break;
        case 16: hipLaunchKernelGGL((sig_combine_kernel<T, T, 16>), grid, block, 0, st, sh, rs, a, b, out); break;
        default: hipLaunchKernelGGL((sig_combine_kernel<T, T, 0>), grid, block, 0, st, sh, rs, a, b, out); break;
    }
    return hipGetLastError();
}

// The word at index i of level k = K (or k_runtime beyond the depths unrolled) of a^{-1} [x] b, for a signature a: the inverse's scalar at a
// word is that of the reversed word of a, negated for odd lengths (section 5.4), so no inverse is formed.  rev is the reversal of the
// prefix of j letters: taking its leading letter off leaves that of j - 1.  Terms and their order are those of product_word.
template <typename T, int K>
__device__ __forceinline__ T interval_word(const T *a, const T *b, uint32_t i, int k_runtime, uint32_t d)
{
    const int k = K > 0 ? K : k_runtime;
    constexpr int kRoom = K > 0 ? K : SIG_MAX_DEPTH;
    uint32_t rev = 0, rest = i, off[kRoom + 1], pw[kRoom + 1];
    pw[0] = 1;
    off[0] = 0;
#pragma unroll
    for (int j = 1; j <= k; ++j) {
        pw[j] = pw[j - 1] * d;
        off[j] = j == 1 ? 0 : off[j - 1] + pw[j - 1];
        rev = rev * d + rest % d;
        rest /= d;
    }
    T x[kRoom], y[kRoom];
    const T whole = a[off[k] + rev], own = b[off[k] + i];
    uint32_t suffix = 0;
#pragma unroll
    for (int j = k - 1; j >= 1; --j) {
        const uint32_t letter = rev / pw[j];   // letter j + 1
        rev -= letter * pw[j];
        suffix += letter * pw[k - 1 - j];
        x[j] = a[off[j] + rev];
        y[j] = b[off[k - j] + suffix];
    }
    T acc = (k & 1 ? -whole : whole) + own;
#pragma unroll
    for (int j = k - 1; j >= 1; --j) acc += (j & 1 ? -x[j] : x[j]) * y[j];
    return acc;
}

// out[p] = a[p]^{-1} [x] b[p], a thread per word; D: the channel count as a constant, or 0.
template <typename T, int D>
__global__ void __launch_bounds__(256)
sig_interval_kernel(Shape sh, int64_t a_stride, int64_t b_stride, int64_t out_stride, const T *__restrict__ a, const T *__restrict__ b,
                    T *__restrict__ out)
{
    const uint32_t d = D > 0 ? uint32_t(D) : uint32_t(sh.d), S = uint32_t(sh.S);
    for (int64_t p = blockIdx.y; p < sh.B; p += gridDim.y) {
        const T *ap = a + p * a_stride, *bp = b + p * b_stride;
        for (uint32_t e = blockIdx.x * 256 + threadIdx.x; e < S; e += gridDim.x * 256) {
            int k = 1;
            uint32_t first = 0;
            for (uint32_t size = d; e - first >= size; size *= d, ++k) first += size;
            const uint32_t i = e - first;
            T v;
            switch (k) {
                case 1: v = interval_word<T, 1>(ap, bp, i, 1, d); break;
                case 2: v = interval_word<T, 2>(ap, bp, i, 2, d); break;
                case 3: v = interval_word<T, 3>(ap, bp, i, 3, d); break;
                case 4: v = interval_word<T, 4>(ap, bp, i, 4, d); break;
                case 5: v = interval_word<T, 5>(ap, bp, i, 5, d); break;
                case 6: v = interval_word<T, 6>(ap, bp, i, 6, d); break;
                case 7: v = interval_word<T, 7>(ap, bp, i, 7, d); break;
                case 8: v = interval_word<T, 8>(ap, bp, i, 8, d); break;
                case 9: v = interval_word<T, 9>(ap, bp, i, 9, d); break;
                default: v = interval_word<T, 0>(ap, bp, i, k, d); break;
            }
            out[p * out_stride + e] = v;
        }
    }
}

template <typename T>
hipError_t launch_interval(const Shape &sh, const T *a, int64_t a_stride, const T *b, int64_t b_stride, T *out, int64_t out_stride,
                           hipStream_t st)
{
    const dim3 grid(unsigned((sh.S + 255) / 256 < 4096 ? (sh.S + 255) / 256 : 4096), unsigned(sh.B < 65535 ? sh.B : 65535));
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, sh, a_stride, b_stride, out_stride, a, b, out);
        return hipGetLastError();
    };
    switch (sh.d) {
        case 2: return go(sig_interval_kernel<T, 2>);
        case 3: return go(sig_interval_kernel<T, 3>);
        case 4: return go(sig_interval_kernel<T, 4>);
        case 5: return go(sig_interval_kernel<T, 5>);
        case 6: return go(sig_interval_kernel<T, 6>);
        case 7: return go(sig_interval_kernel<T, 7>);
        case 8: return go(sig_interval_kernel<T, 8>);
    }
    return go(sig_interval_kernel<T, 0>);
}

}  // namespace

hipError_t launch_interval_f32(const Shape &sh, const float *a, int64_t a_stride, const float *b, int64_t b_stride, float *out,
                               int64_t out_stride, hipStream_t st)
{
    return launch_interval<float>(sh, a, a_stride, b, b_stride, out, out_stride, st);
}

hipError_t launch_interval_f64(const Shape &sh, const double *a, int64_t a_stride, const double *b, int64_t b_stride, double *out,
                               int64_t out_stride, hipStream_t st)
{
    return launch_interval<double>(sh, a, a_stride, b, b_stride, out, out_stride, st);
}

bool combine_supported(const Shape &sh) { return sh.S < (int64_t(1) << 31); }

hipError_t launch_combine_f32(const Shape &sh, const float *a, const float *b, float *out, hipStream_t st,
                              const int64_t *strides)
{
    return launch_combine<float>(sh, a, b, out, st, strides);
}

hipError_t launch_combine_f64(const Shape &sh, const double *a, const double *b, double *out, hipStream_t st,
                              const int64_t *strides)
{
    return launch_combine<double>(sh, a, b, out, st, strides);
}

}  // namespace sig
