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

// a^{-1} [x] b for signatures a: the inverse's scalar at a word is that of the reversed word of a, negated for odd lengths (section 5.4),
// so no inverse is formed.  What bounds it is the reading of a: in the order of the words neighbours lie d^(k-1) scalars apart in a, and
// each fetches a line of its own.  So a thread takes W words that differ in their last letter only, and the threads are counted by
// these groups, the E last letters of the prefix, then its F first ones in reverse: a wavefront writes and reads b in runs of d^(E+1) words,
// and reads a in runs of up to d^F scalars.  Neighbouring workgroups go to one XCD, so that the rest of a line is found in its L2.
// Measured: a query in us, the host's 6.5 included (with a kept inverse through sig_combine 10.7 of it | a word per thread in the order of
// the words | this): 512 paths, d = 5, N = 5 10.7 | 25 | 9.6; 256, d = 6, N = 5 10.5 | 30 | 10.3, fp64 14.8 | 30 | 14.3; 32, d = 16, N = 4 11 | 30 | 9.3,
// fp64 11.5 | 20 | 12.9; 8, d = 9, N = 6 37 | 70 | 38; 4, d = 2, N = 15 10.6 | 35 | 8.2; 32, d = 4, N = 4 11.5 | 6.8 | 6.9.
struct IntervalGrid {
    int F, E;                             // letters, where the channel count is not a constant
    uint32_t groups;                      // threads for the words of a prefix
    uint32_t blocks[SIG_MAX_DEPTH + 1];   // workgroups of a level, a multiple of 8
};

constexpr int interval_first(int d) { return d == 2 ? 4 : d == 3 ? 3 : d <= 8 ? 2 : 1; }
constexpr int interval_last(int d) { return d == 2 ? 3 : d == 3 ? 2 : d <= 8 ? 1 : 0; }

// The `digits` digits of v in reverse; UNROLL: at most so many of them, or 1 where they are a run-time value.
template <int UNROLL>
__device__ __forceinline__ uint32_t reversed_word(uint32_t v, int digits, uint32_t d)
{
    uint32_t r = 0;
#pragma unroll(UNROLL)
    for (int i = 0; i < digits; ++i) {
        const uint32_t q = v / d;
        r = r * d + (v - q * d);
        v = q;
    }
    return r;
}

// The words of thread t (of d^(k-1) groups) in level k = K, or k_runtime beyond the depths unrolled.
template <typename T, int D, int W, int K>
__device__ __forceinline__ void interval_words(const Shape &sh, const IntervalGrid &grid, int k_runtime, uint32_t t, const T *a, const T *b, T *out)
{
    const uint32_t d = D > 0 ? uint32_t(D) : uint32_t(sh.d);
    constexpr int kUnroll = K > 0 ? K : 1;
    const int k = K > 0 ? K : k_runtime, letters = k - 1;
    const auto pw = [&](int j) {
        if constexpr (D > 0 && K > 0) {
            uint32_t p = 1;
            for (int i = 0; i < j; ++i) p *= uint32_t(D);
            return p;
        } else {
            return uint32_t(sh.pw[j]);
        }
    };
    const auto off = [&](int j) { return uint32_t(sh.off[j]); };
    const int first = D > 0 ? interval_first(D) : grid.F, last = D > 0 ? interval_last(D) : grid.E;
    const int F = first < letters ? first : letters, E = last < letters - F ? last : letters - F;
    uint32_t c0 = 0;
    if constexpr (W != D) {
        c0 = t % grid.groups * W;
        t /= grid.groups;
    }
    const uint32_t v = t % pw(E);
    t /= pw(E);
    const uint32_t u_rev = t % pw(F), m = t / pw(F);
    const uint32_t prefix = reversed_word<kUnroll>(u_rev, F, d) * pw(letters - F) + m * pw(E) + v;
    const uint32_t rev = reversed_word<kUnroll>(v, E, d) * pw(letters - E) + reversed_word<kUnroll>(m, letters - F - E, d) * pw(F) + u_rev;
    // the words of the prefix, moved as a vector unless some are missing
    typedef Siblings<T, W> V;
    const bool whole_v = W == D || c0 + W <= d;
    const auto words = [&](const T *p) {
        if (whole_v) return *reinterpret_cast<const V *>(p + c0);
        V r;
#pragma unroll
        for (int c = 0; c < W; ++c) r.v[c] = p[c0 + c < d ? c0 + c : d - 1];
        return r;
    };
    V acc = words(b + off(k) + prefix * d);
    {
        const uint32_t at = off(k) + rev;
        V own;
#pragma unroll
        for (int c = 0; c < W; ++c) {
            own.v[c] = a[at + (whole_v || c0 + c < d ? c0 + c : d - 1) * pw(letters)];
            if (k & 1) own.v[c] = -own.v[c];
        }
        acc = own + acc;
    }
#pragma unroll(kUnroll)
    for (int j = letters; j >= 1; --j) {
        const T x = a[off(j) + rev % pw(j)];
        acc += (j & 1 ? -x : x) * words(b + off(k - j) + prefix % pw(letters - j) * d);
    }
    T *o = out + off(k) + prefix * d + c0;
    if (whole_v) {
        *reinterpret_cast<V *>(o) = acc;
    } else {
#pragma unroll
        for (int c = 0; c < W; ++c)
            if (c0 + c < d) o[c] = acc.v[c];
    }
}

// A workgroup takes words of one level of one path or several; D: the channel count as a constant, or 0.
template <typename T, int D, int W>
__global__ void __launch_bounds__(256)
sig_interval_kernel(Shape sh, IntervalGrid grid, int64_t a_stride, int64_t b_stride, int64_t out_stride, const T *__restrict__ a,
                    const T *__restrict__ b, T *__restrict__ out)
{
    uint32_t block = blockIdx.x;
    int k = sh.N;
    for (; k > 1 && block >= grid.blocks[k]; --k) block -= grid.blocks[k];
    block = block % 8 * (grid.blocks[k] / 8) + block / 8;   // neighbours on one XCD, whose L2 then holds whole lines
    const uint32_t e = block * 256 + threadIdx.x, size = uint32_t(sh.pw[k - 1]) * grid.groups, p = e / size, t = e - p * size;
    if (int64_t(p) >= sh.B) return;
    const T *ap = a + int64_t(p) * a_stride, *bp = b + int64_t(p) * b_stride;
    T *op = out + int64_t(p) * out_stride;
    switch (k) {
        case 1: return interval_words<T, D, W, 1>(sh, grid, 1, t, ap, bp, op);
        case 2: return interval_words<T, D, W, 2>(sh, grid, 2, t, ap, bp, op);
        case 3: return interval_words<T, D, W, 3>(sh, grid, 3, t, ap, bp, op);
        case 4: return interval_words<T, D, W, 4>(sh, grid, 4, t, ap, bp, op);
        case 5: return interval_words<T, D, W, 5>(sh, grid, 5, t, ap, bp, op);
        case 6: return interval_words<T, D, W, 6>(sh, grid, 6, t, ap, bp, op);
        case 7: return interval_words<T, D, W, 7>(sh, grid, 7, t, ap, bp, op);
        case 8: return interval_words<T, D, W, 8>(sh, grid, 8, t, ap, bp, op);
        case 9: return interval_words<T, D, W, 9>(sh, grid, 9, t, ap, bp, op);
    }
    if constexpr (D == 2) {   // (2048 paths, N = 10: 25.6 | 21.4 us)
        switch (k) {
            case 10: return interval_words<T, D, W, 10>(sh, grid, 10, t, ap, bp, op);
            case 11: return interval_words<T, D, W, 11>(sh, grid, 11, t, ap, bp, op);
            case 12: return interval_words<T, D, W, 12>(sh, grid, 12, t, ap, bp, op);
        }
    }
    interval_words<T, D, W, 0>(sh, grid, k, t, ap, bp, op);
}

template <typename T, int D, int W>
hipError_t launch_interval_d(Shape sh, const T *a, int64_t a_stride, const T *b, int64_t b_stride, T *out, int64_t out_stride, hipStream_t st)
{
    IntervalGrid grid = {};
    grid.F = interval_first(sh.d);
    grid.E = interval_last(sh.d);
    grid.groups = uint32_t((sh.d + W - 1) / W);
    // threads are counted in 32 bits: so many paths to a launch (one has less than 2^31)
    const int64_t paths = sh.B, most = ((int64_t(1) << 31) - 1) / (sh.pw[sh.N - 1] * grid.groups);
    for (int64_t p = 0; p < paths; p += sh.B) {
        sh.B = paths - p < most ? paths - p : most;
        int64_t blocks = 0;
        for (int k = 1; k <= sh.N; ++k) {
            grid.blocks[k] = uint32_t((sh.B * sh.pw[k - 1] * grid.groups + 2047) / 2048 * 8);
            blocks += grid.blocks[k];
        }
        hipLaunchKernelGGL((sig_interval_kernel<T, D, W>), dim3(unsigned(blocks)), dim3(256), 0, st, sh, grid, a_stride, b_stride, out_stride,
                           a + p * a_stride, b + p * b_stride, out + p * out_stride);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

// W: all words of a prefix, in fp64 two from six channels on where that divides (32, d = 16, N = 4: 2 | 4 | 8 | 16 words 12.9 | 15 | 18 | 18 us;
// fp32 16 | 4 words 9.3 | 13.5; 64 paths, d = 8, N = 5 8 | 4 words 9.2 | 19.6).
template <typename T>
hipError_t launch_interval(const Shape &sh, const T *a, int64_t a_stride, const T *b, int64_t b_stride, T *out, int64_t out_stride,
                           hipStream_t st)
{
    constexpr bool f32 = sizeof(T) == 4;
    switch (sh.d) {
        case 2: return launch_interval_d<T, 2, 2>(sh, a, a_stride, b, b_stride, out, out_stride, st);
        case 3: return launch_interval_d<T, 3, 3>(sh, a, a_stride, b, b_stride, out, out_stride, st);
        case 4: return launch_interval_d<T, 4, 4>(sh, a, a_stride, b, b_stride, out, out_stride, st);
        case 5: return launch_interval_d<T, 5, 5>(sh, a, a_stride, b, b_stride, out, out_stride, st);
        case 6: return launch_interval_d<T, 6, f32 ? 6 : 2>(sh, a, a_stride, b, b_stride, out, out_stride, st);
        case 7: return launch_interval_d<T, 7, 7>(sh, a, a_stride, b, b_stride, out, out_stride, st);
        case 8: return launch_interval_d<T, 8, f32 ? 8 : 2>(sh, a, a_stride, b, b_stride, out, out_stride, st);
        case 16: return launch_interval_d<T, 16, f32 ? 16 : 2>(sh, a, a_stride, b, b_stride, out, out_stride, st);
    }
    return launch_interval_d<T, 0, 4>(sh, a, a_stride, b, b_stride, out, out_stride, st);
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
