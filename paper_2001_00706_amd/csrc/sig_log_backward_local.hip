// The gradient through the logarithm where a truncated element fits the LDS of a compute unit: whole signatures of the channel counts that
// have no kernel of their own in sig_log_backward.hip (3, 5, 6, 7; 9 to 16 at depth 3), and the last steps of those that are too large,
// whose cotangent loses its top level at every step (3 to 16; the recurrences are there).  A workgroup per signature; step m needs
//     G_{m+1}[v] = sum_u x[u] G_m[u v],   gx[u] += c_m G_m[u] + sum_v G_m[u v] R_{m+1}[v]    at levels 1..n-1 of G_m's n
// which are dot products along the flat order: the words u v of k + l letters follow one another.  Level l has d^l outputs of each kind with
// about as many terms in all as any other level, so each of its dot products is taken by as many lanes as give every thread one,
// and they meet by lane exchanges.  One barrier a step, none within; d and n are constants, so all places fold.
//
// What bounds it is the latency of the LDS reads of a step, 1 to 2 us.  Before (a workgroup that walks a matrix at a time with two barriers
// a pass, or two launches a step) | now, us: 256 signatures of d = 6, N = 4 21.5 | 7.6, 2000 of d = 5, N = 5 148 | 36, 1500 of d = 7, N = 4 73 | 18,
// 1024 of d = 3, N = 6 50 | 14; the last four of six steps of 32 at d = 5, N = 7 37 | 12, of the whole gradient 105 | 80.
#include "sig_internal.h"

#include <type_traits>

namespace sig {
namespace {

constexpr int64_t ll_pow(int d, int k)
{
    int64_t p = 1;
    for (int i = 0; i < k; ++i) p *= d;
    return p;
}
constexpr int ll_off(int d, int k)   // offset of level k (1-based); ll_off(d, k + 1) scalars up to level k
{
    int64_t off = 0;
    for (int j = 1; j < k; ++j) off += ll_pow(d, j);
    return int(off);
}
constexpr int ll_r_at(int d, int n, int k)   // place of the R with k levels among those with 1, 2, .. levels
{
    int at = 0;
    for (int i = 1; i < k; ++i) at += ll_off(d, i + 1);
    return at;
}

// LEVELS of the first cotangent.  LDS: x (LEVELS - 1 levels) | R with 1 .. LEVELS - 1 levels | G, twice | gx.
template <int D, int LEVELS>
struct LocalShape {
    static constexpr int kS = ll_off(D, LEVELS + 1), kLow = ll_off(D, LEVELS);
    static constexpr int kAtR = kLow, kAtG = kAtR + ll_r_at(D, LEVELS, LEVELS), kAtG2 = kAtG + kS, kAtGx = kAtG2 + kLow, kScalars = kAtGx + kS;
    static constexpr int NT = kS <= 800 ? 256 : 512;
};

template <int LANES, typename T>
__device__ __forceinline__ T ll_sum(T v)
{
#pragma unroll
    for (int m = 1; m < LANES; m *= 2) v += __shfl_xor(v, m);
    return v;
}

constexpr int ll_lanes(int outputs, int terms, int threads)
{
    int lanes = 1;
    while (lanes < 64 && 2 * lanes * outputs <= threads && 2 * lanes <= terms) lanes *= 2;
    return lanes;
}

// One step at level L of the outputs; G has n levels.
template <typename T, int D, int n, int L, int NT>
__device__ __forceinline__ void ll_level(int tid, const T *x, const T *R, const T *G, T *Gn, T *gx, T c)
{
    constexpr int kOut = int(ll_pow(D, L)), kTerms = ll_off(D, n - L + 1), kLanes = ll_lanes(2 * kOut, kTerms, NT), kGroups = NT / kLanes;
    const int sub = tid % kLanes;
    for (int o = tid / kLanes; o < 2 * kOut; o += kGroups) {
        const bool left = o >= kOut;   // gx, the sum over suffixes
        const int w = left ? o - kOut : o;
        T acc = T(0);
        const auto level = [&](auto k_) {
            constexpr int k = decltype(k_)::value;
            if constexpr (k <= n - L) {
                constexpr int count = int(ll_pow(D, k)), at = ll_off(D, k), from = ll_off(D, k + L);
                const T *a = (left ? R : x) + at, *g = G + from + (left ? w * count : w);
                const int step = left ? 1 : kOut;
                T part = T(0);
#pragma unroll 8
                for (int i = sub; i < count; i += kLanes) part += a[i] * g[i * step];
                acc += part;
            }
        };
        level(std::integral_constant<int, 1>{});
        level(std::integral_constant<int, 2>{});
        level(std::integral_constant<int, 3>{});
        level(std::integral_constant<int, 4>{});
        level(std::integral_constant<int, 5>{});
        level(std::integral_constant<int, 6>{});
        level(std::integral_constant<int, 7>{});
        acc = ll_sum<kLanes>(acc);
        if (sub == 0) {
            const int to = ll_off(D, L) + w;
            if (left)
                gx[to] += acc + c * G[to];
            else
                Gn[to] = acc;
        }
    }
    if constexpr (L + 1 < n) ll_level<T, D, n, L + 1, NT>(tid, x, R, G, Gn, gx, c);
}

// Steps from the one whose cotangent has n levels on; c of the last (one level) is cs[1].
template <typename T, int D, int n, int LEVELS, int NT>
__device__ __forceinline__ void ll_steps(int tid, const T *x, const T *Rs, T *G, T *Gn, T *gx, const T *cs)
{
    if constexpr (n >= 2) {
        const T c = cs[n];
        ll_level<T, D, n, 1, NT>(tid, x, Rs + ll_r_at(D, LEVELS, n - 1), G, Gn, gx, c);
        for (int i = ll_off(D, n) + tid; i < ll_off(D, n + 1); i += NT) gx[i] += c * G[i];
        __syncthreads();
        ll_steps<T, D, n - 1, LEVELS, NT>(tid, x, Rs, Gn, G, gx, cs);
    } else {
        if (tid < D) gx[tid] += cs[1] * G[tid];
        __syncthreads();
    }
}

// R_m = c_m x + x R_{m+1}, k levels of it from the k - 1 of the one before.
template <typename T, int D, int LEVELS, int k, int NT>
__device__ __forceinline__ void ll_make_r(int tid, const T *x, T *Rs, const T *cs)
{
    if constexpr (k < LEVELS) {
        T *out = Rs + ll_r_at(D, LEVELS, k);
        const T *next = Rs + ll_r_at(D, LEVELS, k - 1);
        const auto level = [&](auto j_) {
            constexpr int j = decltype(j_)::value;   // letters
            if constexpr (j <= k) {
                for (int w = tid; w < int(ll_pow(D, j)); w += NT) {
                    T acc = cs[k] * x[ll_off(D, j) + w];
#pragma unroll
                    for (int i = j - 1; i >= 1; --i) {   // letters of the prefix, the longest first
                        const int after = int(ll_pow(D, j - i));
                        acc += x[ll_off(D, i) + w / after] * next[ll_off(D, j - i) + w % after];
                    }
                    out[ll_off(D, j) + w] = acc;
                }
            }
        };
        level(std::integral_constant<int, 1>{});
        level(std::integral_constant<int, 2>{});
        level(std::integral_constant<int, 3>{});
        level(std::integral_constant<int, 4>{});
        level(std::integral_constant<int, 5>{});
        level(std::integral_constant<int, 6>{});
        level(std::integral_constant<int, 7>{});
        __syncthreads();
        ll_make_r<T, D, LEVELS, k + 1, NT>(tid, x, Rs, cs);
    }
}

// WHOLE: signatures of depth LEVELS, r is not read, gx is written.  Otherwise the steps from the one on whose cotangent g has LEVELS levels:
// r holds the R with 1, 2, .. levels one after the other, and gx is added to.
template <typename T, int D, int LEVELS, bool WHOLE>
__global__ void __launch_bounds__((LocalShape<D, LEVELS>::NT))
log_bwd_local_kernel(int N, int64_t S, const T *__restrict__ x_g, const T *__restrict__ r_g, int64_t r_stride, const T *__restrict__ g_g,
                     int64_t g_stride, T *__restrict__ gx_g)
{
    using LS = LocalShape<D, LEVELS>;
    constexpr int NT = LS::NT;
    extern __shared__ __align__(16) unsigned char smem[];
    T *x = reinterpret_cast<T *>(smem), *Rs = x + LS::kAtR, *G = x + LS::kAtG, *G2 = x + LS::kAtG2, *gx = x + LS::kAtGx;
    __shared__ T cs[LEVELS + 1];   // c_m by the levels of G_m, N - m + 1
    const int tid = threadIdx.x;
    const int64_t row = blockIdx.x;
    x_g += row * S;
    g_g += row * g_stride;
    gx_g += row * S;
    if (tid >= 1 && tid <= LEVELS) {
        const int m = N - tid + 1;
        cs[tid] = (m & 1 ? T(1) : T(-1)) / T(m);
    }
    for (int i = tid; i < LS::kLow; i += NT) x[i] = x_g[i];
    for (int i = tid; i < LS::kS; i += NT) {
        G[i] = g_g[i];
        gx[i] = WHOLE ? T(0) : gx_g[i];
    }
    if constexpr (!WHOLE) {
        r_g += row * r_stride;
        for (int i = tid; i < ll_r_at(D, LEVELS, LEVELS); i += NT) Rs[i] = r_g[i];
    }
    __syncthreads();
    if constexpr (WHOLE) {
        if (tid < D) Rs[tid] = cs[1] * x[tid];
        __syncthreads();
        ll_make_r<T, D, LEVELS, 2, NT>(tid, x, Rs, cs);
    }
    ll_steps<T, D, LEVELS, LEVELS, NT>(tid, x, Rs, G, G2, gx, cs);
    for (int i = tid; i < LS::kS; i += NT) gx_g[i] = gx[i];
}

template <typename T, int D, int LEVELS, bool WHOLE>
hipError_t launch_local(const Shape &sh, const T *x, const T *r, int64_t r_stride, const T *g, int64_t g_stride, T *gx, hipStream_t st)
{
    using LS = LocalShape<D, LEVELS>;
    constexpr int kBytes = LS::kScalars * int(sizeof(T));
    static_assert(kBytes <= 158 * 1024);
    const auto kernel = log_bwd_local_kernel<T, D, LEVELS, WHOLE>;
    if (kBytes > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
        if (e != hipSuccess) return e;
    }
    // A grid has less than 2^32 threads.  (Workgroups that go on to further signatures would keep the places worked out for all of them in
    // registers: 1024 of d = 3, N = 6 took 34 us instead of 14.)
    constexpr int64_t kMost = int64_t(1) << 22;
    for (int64_t first = 0; first < sh.B; first += kMost) {
        const int64_t count = sh.B - first < kMost ? sh.B - first : kMost;
        hipLaunchKernelGGL(kernel, dim3(unsigned(count)), dim3(LS::NT), kBytes, st, sh.N, sh.S, x + first * sh.S, WHOLE ? r : r + first * r_stride,
                           r_stride, g + first * g_stride, g_stride, gx + first * sh.S);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

}  // namespace

int log_backward_local_levels(int d)
{
    switch (d) {
        case 3: return 7;
        case 4: return 5;
        case 5: return 5;
        case 6: return 4;
        case 7: return 4;
        case 8: return 4;
    }
    return d >= 9 && d <= 16 ? 3 : 0;
}

namespace {

// f of the channel count as a constant, 9 to 16
template <typename F>
hipError_t with_many_channels(int d, F f)
{
    switch (d) {
        case 9: return f(std::integral_constant<int, 9>{});
        case 10: return f(std::integral_constant<int, 10>{});
        case 11: return f(std::integral_constant<int, 11>{});
        case 12: return f(std::integral_constant<int, 12>{});
        case 13: return f(std::integral_constant<int, 13>{});
        case 14: return f(std::integral_constant<int, 14>{});
        case 15: return f(std::integral_constant<int, 15>{});
        case 16: return f(std::integral_constant<int, 16>{});
    }
    return hipErrorNotSupported;
}

}  // namespace

template <typename T>
hipError_t launch_log_backward_whole(const Shape &sh, const T *x, const T *g, T *gx, hipStream_t st)
{
    const T *none = nullptr;
    if constexpr (sizeof(T) == 4) {   // 109 and 87 KB
        if (sh.d == 3 && sh.N == 8) return launch_local<T, 3, 8, true>(sh, x, none, 0, g, sh.S, gx, st);
        if (sh.d == 6 && sh.N == 5) return launch_local<T, 6, 5, true>(sh, x, none, 0, g, sh.S, gx, st);
    }
    if (sh.d > 8 && sh.N == 3)
        return with_many_channels(sh.d, [&](auto d) { return launch_local<T, decltype(d)::value, 3, true>(sh, x, none, 0, g, sh.S, gx, st); });
    if (sh.d > 8 || sh.N > 9) return hipErrorNotSupported;
    switch (sh.d * 10 + sh.N) {
        case 33: return launch_local<T, 3, 3, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 34: return launch_local<T, 3, 4, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 35: return launch_local<T, 3, 5, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 36: return launch_local<T, 3, 6, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 37: return launch_local<T, 3, 7, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 53: return launch_local<T, 5, 3, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 54: return launch_local<T, 5, 4, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 55: return launch_local<T, 5, 5, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 63: return launch_local<T, 6, 3, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 64: return launch_local<T, 6, 4, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 73: return launch_local<T, 7, 3, true>(sh, x, none, 0, g, sh.S, gx, st);
        case 74: return launch_local<T, 7, 4, true>(sh, x, none, 0, g, sh.S, gx, st);
    }
    return hipErrorNotSupported;
}

template <typename T>
hipError_t launch_log_backward_tail(const Shape &sh, const T *x, const T *r, int64_t r_stride, const T *g, int64_t g_stride, T *gx,
                                    hipStream_t st)
{
    switch (sh.d) {
        case 3: return launch_local<T, 3, 7, false>(sh, x, r, r_stride, g, g_stride, gx, st);
        case 4: return launch_local<T, 4, 5, false>(sh, x, r, r_stride, g, g_stride, gx, st);
        case 5: return launch_local<T, 5, 5, false>(sh, x, r, r_stride, g, g_stride, gx, st);
        case 6: return launch_local<T, 6, 4, false>(sh, x, r, r_stride, g, g_stride, gx, st);
        case 7: return launch_local<T, 7, 4, false>(sh, x, r, r_stride, g, g_stride, gx, st);
        case 8: return launch_local<T, 8, 4, false>(sh, x, r, r_stride, g, g_stride, gx, st);
    }
    return with_many_channels(
        sh.d, [&](auto d) { return launch_local<T, decltype(d)::value, 3, false>(sh, x, r, r_stride, g, g_stride, gx, st); });
}

template hipError_t launch_log_backward_whole<float>(const Shape &, const float *, const float *, float *, hipStream_t);
template hipError_t launch_log_backward_whole<double>(const Shape &, const double *, const double *, double *, hipStream_t);
template hipError_t launch_log_backward_tail<float>(const Shape &, const float *, const float *, int64_t, const float *, int64_t, float *, hipStream_t);
template hipError_t launch_log_backward_tail<double>(const Shape &, const double *, const double *, int64_t, const double *, int64_t, double *,
                                                     hipStream_t);

}  // namespace sig
