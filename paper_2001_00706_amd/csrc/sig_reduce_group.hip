// Products of several consecutive signatures in one launch (fp32 and fp64, 2 to 8 channels): the rounds of a product tree that is too large for
// a workgroup.
//
// A round of the tree halves the count and is a launch; the last ones are little but the launch, 3.3 us each.  A product is formed
// from left to right for the words below any prefix by themselves: [P C](w) = P(w) + C(w) + sum over w = u v of P(u) C(v).  So a thread keeps
// the running product at a word of N - 1 letters, its prefixes and its children in registers, and a step needs the next signature only, whose
// levels up to N - 1 the workgroup stages in LDS while the step before is formed.  Eight signatures one after the other round the running
// sums seven times where three rounds do it three times (1.1 to 1.4 times the error): what the additions round off is kept beside them
// (the error of an addition by six more, as Knuth's and Moller's).
// One path of 65537 points, d = 4, N = 6: 1024 signatures in 4 launches of 4 to 8 us, 24 in all, instead of 10 that took 45.
#include "sig_internal.h"
#include "sig_lane_ops.h"
#include "sig_tile_common.h"

namespace sig {
namespace {

template <typename T, int D, int N>
struct GroupShape {
    static constexpr int letters_of_u()
    {
        int y = 0;
        while (tl_pow(D, N - 1 - y) > 512) ++y;
        return y;
    }
    static constexpr int Y = letters_of_u();                                  // letters that a workgroup's words share
    static constexpr int kWords = int(tl_pow(D, N - 1 - Y)), kThreads = (kWords + 63) / 64 * 64;
    static constexpr int64_t kGroups = tl_pow(D, Y), kLow = tl_off(D, N);     // workgroups of a product; scalars of the levels up to N - 1
    static constexpr int kLoads = int((kLow + kThreads - 1) / kThreads);      // of a thread and signature
    static constexpr bool kServed = 2 * kLow * int(sizeof(T)) <= 48 * 1024 && kLoads <= 16;
};

// sum += v, what the addition rounds off kept in `lost`
template <typename T>
__device__ __forceinline__ void add_keeping(T &sum, T &lost, T v)
{
    const T t = sum + v, part = t - sum;
    lost += (sum - (t - part)) + (v - part);
    sum = t;
}

// ... and in the end: a sum that is infinite has lost what is no number.
template <typename T>
__device__ __forceinline__ T with_lost(T sum, T lost)
{
    const T t = sum + lost;
    return t == t ? t : sum;
}

// to[r] = the product of the signatures r R .. r R + R - 1 of `from`, R >= 2
template <typename T, int D, int N>
__global__ void __launch_bounds__((GroupShape<T, D, N>::kThreads))
sig_reduce_group_kernel(int R, const T *__restrict__ from, T *__restrict__ to)
{
    using GS = GroupShape<T, D, N>;
    constexpr int64_t kS = tl_off(D, N + 1);
    constexpr int kLow = int(GS::kLow), NT = GS::kThreads;
    __shared__ __align__(16) T low[2][kLow];
    const int tid = threadIdx.x;
    const int64_t product = blockIdx.x / unsigned(GS::kGroups);
    const int u = int(blockIdx.x - unsigned(product) * unsigned(GS::kGroups));
    const bool there = tid < GS::kWords;
    const int w = u * GS::kWords + (there ? tid : 0);
    const T *c = from + product * R * kS;

    int wk[N];   // the word's prefix of k letters
    T p[N], leaf[D];
    {
        int rest = w;
#pragma unroll
        for (int k = N - 1; k >= 1; --k) {
            wk[k] = rest;
            p[k] = c[tl_off(D, k) + rest];
            rest /= D;
        }
    }
#pragma unroll
    for (int j = 0; j < D; ++j) leaf[j] = c[tl_off(D, N) + int64_t(w) * D + j];
    T p_lost[N] = {}, leaf_lost[D] = {};
    T staged[GS::kLoads], leaf_next[D];
    const auto fetch = [&](const T *next) {
#pragma unroll
        for (int i = 0; i < GS::kLoads; ++i) {
            const int e = tid + i * NT;
            staged[i] = next[e < kLow ? e : kLow - 1];
        }
#pragma unroll
        for (int j = 0; j < D; ++j) leaf_next[j] = next[tl_off(D, N) + int64_t(w) * D + j];
    };
    fetch(c + kS);
    for (int r = 1; r < R; ++r) {
        T *l = low[r & 1];   // last read two steps ago: a barrier lies between
#pragma unroll
        for (int i = 0; i < GS::kLoads; ++i) {
            const int e = tid + i * NT;
            if (e < kLow) l[e] = staged[i];
        }
        T own[D];
#pragma unroll
        for (int j = 0; j < D; ++j) own[j] = leaf_next[j];
        lds_barrier();
        if (r + 1 < R) fetch(c + (r + 1) * kS);
#pragma unroll
        for (int i = 1; i < N; ++i) {   // the first i letters from the left
            const int at = int(tl_off(D, N - i)) + wk[N - 1] % int(tl_pow(D, N - 1 - i)) * D;
#pragma unroll
            for (int j = 0; j < D; ++j) own[j] += p[i] * l[at + j];
        }
#pragma unroll
        for (int j = 0; j < D; ++j) add_keeping(leaf[j], leaf_lost[j], own[j]);
#pragma unroll
        for (int k = N - 1; k >= 1; --k) {
            T sum = l[tl_off(D, k) + wk[k]];
#pragma unroll
            for (int i = 1; i < k; ++i) sum += p[i] * l[tl_off(D, k - i) + wk[k] % int(tl_pow(D, k - i))];
            add_keeping(p[k], p_lost[k], sum);
        }
    }
    if (!there) return;
    T *out = to + product * kS;
#pragma unroll
    for (int j = 0; j < D; ++j) out[tl_off(D, N) + int64_t(w) * D + j] = with_lost(leaf[j], leaf_lost[j]);
#pragma unroll
    for (int k = N - 1; k >= 1; --k)   // by the first word below
        if (wk[N - 1] % int(tl_pow(D, N - 1 - k)) == 0) out[tl_off(D, k) + wk[k]] = with_lost(p[k], p_lost[k]);
}

template <typename T, int D, int N>
hipError_t launch_dn(int64_t products, int R, const T *from, T *to, hipStream_t st)
{
    using GS = GroupShape<T, D, N>;
    if constexpr (GS::kServed) {
        if (!grid_holds(products * GS::kGroups, GS::kThreads)) return hipErrorNotSupported;
        hipLaunchKernelGGL((sig_reduce_group_kernel<T, D, N>), dim3(unsigned(products * GS::kGroups)), dim3(GS::kThreads), 0, st, R, from, to);
        return hipGetLastError();
    }
    return hipErrorNotSupported;
}

template <typename T, int D>
hipError_t launch_d(int N, int64_t products, int R, const T *from, T *to, hipStream_t st)
{
    switch (N) {
        case 3: return launch_dn<T, D, 3>(products, R, from, to, st);
        case 4: return launch_dn<T, D, 4>(products, R, from, to, st);
        case 5: return launch_dn<T, D, 5>(products, R, from, to, st);
        case 6: return launch_dn<T, D, 6>(products, R, from, to, st);
        case 7: return launch_dn<T, D, 7>(products, R, from, to, st);
        case 8: return launch_dn<T, D, 8>(products, R, from, to, st);
    }
    return hipErrorNotSupported;
}

template <typename T>
hipError_t launch(const Shape &sh, int64_t products, int R, const T *from, T *to, hipStream_t st)
{
    switch (sh.d) {
        case 2: return launch_d<T, 2>(sh.N, products, R, from, to, st);
        case 3: return launch_d<T, 3>(sh.N, products, R, from, to, st);
        case 4: return launch_d<T, 4>(sh.N, products, R, from, to, st);
        case 5: return launch_d<T, 5>(sh.N, products, R, from, to, st);
        case 6: return launch_d<T, 6>(sh.N, products, R, from, to, st);
        case 7: return launch_d<T, 7>(sh.N, products, R, from, to, st);
        case 8: return launch_d<T, 8>(sh.N, products, R, from, to, st);
    }
    return hipErrorNotSupported;
}

}  // namespace

hipError_t launch_reduce_group_f32(const Shape &sh, int64_t products, int R, const float *from, float *to, hipStream_t st)
{
    return launch<float>(sh, products, R, from, to, st);
}
hipError_t launch_reduce_group_f64(const Shape &sh, int64_t products, int R, const double *from, double *to, hipStream_t st)
{
    return launch<double>(sh, products, R, from, to, st);
}

}  // namespace sig
