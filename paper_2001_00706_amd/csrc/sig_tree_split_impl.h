// Prefix-tree scan in final mode with a path cut into stretches that share a workgroup (d = 2..8 at N = 3..9, d = 9..16 at N = 3; fp32
// and fp64), for batches that leave the chip idle.
//
// What bounds sig_tree_kernel with few paths is the latency of its chain of increments, 0.25 to 0.3 us each while a SIMD has a
// wavefront or less (a path of 100 points takes 28 us whatever its size).  The product is associative (paper section 5.1), so K threads
// scan a word's K stretches at the same time and the stretches' signatures are joined in log2 K rounds through LDS: those on the
// right leave their signature there, and a thread on the left, which holds all prefixes of its words, multiplies it on
// with reads at the suffixes of its words alone (sig_stretch_ops.h).  All in one launch, nothing in memory.
#ifndef SIG_TREE_SPLIT_IMPL_H_
#define SIG_TREE_SPLIT_IMPL_H_

#include "sig_stretch_ops.h"
#include "sig_tree_impl.h"

namespace sig {
namespace {

constexpr int kSplitTile = 16;              // increments of a stretch staged in LDS at a time
constexpr int kSplitLds = 150 * 1024;       // bytes of LDS a workgroup may take

template <typename T, int D, int N>
struct SplitShape {
    // levels below a thread's word: as in sig_tree_kernel, but one at depth 3, where a thread per letter would be too few
    static constexpr int U = D <= 8 && N >= 4 ? 2 : 1, P = N - U;
    static constexpr int64_t kAllWords = tree_off(D, P + 1) - tree_off(D, P);
    static constexpr int kWords = int(kAllWords < 4096 ? kAllWords : 4096);
    // 16 wavefronts leave 128 registers a lane, enough for a share of up to six channels in fp32
    static constexpr int kThreads = sizeof(T) == 4 && D <= 6 ? 1024 : 512;
    static constexpr int kRow = kSplitTile * D + 1;                      // scalars of a stretch's increments in LDS
    static constexpr int kPerThread = (kSplitTile * D + kWords - 1) / kWords;
};

// One increment (a row of D scalars in LDS) folded into a thread's share, the recurrence of sig_tree_kernel: the coefficients A of its word
// and of the prefixes, B1 and B2 of the words one and two letters longer; cl: the word's letters, rk[m] = 1 / m.
template <typename T, int D, int N, int U>
__device__ __forceinline__ void split_increment(const T *zrow, const int *cl, const T *rk, T *A, T *B1, T *B2)
{
    constexpr int P = N - U;
    // every read is issued before the first is used, as there (and with the same exception; in this kernel d = 7 is 0 to 5 % behind with it,
    // 4 x 400 points, N = 4 20.0 us against 19.0)
    T zl[P + 1], zu[D];
#pragma unroll
    for (int i = 1; i <= P; ++i) zl[i] = zrow[cl[i]];
#pragma unroll
    for (int c = 0; c < D; ++c) zu[c] = zrow[c];
    __builtin_amdgcn_sched_barrier(D == 7 ? 1 : 0);
    // Horner terms along the word: Hn[k] = T^(k)_i for the level i just passed, k > i
    T Hn[N + 2];
    {
        const T zc = zl[1];
#pragma unroll
        for (int k = 2; k <= N; ++k) Hn[k] = fma_t(zc, rk[k], A[1]);
        A[1] += zc;
    }
#pragma unroll
    for (int i = 2; i <= P; ++i) {
        const T zc = zl[i];
        const T a = A[i];
        A[i] = fma_t(Hn[i], zc, a);
#pragma unroll
        for (int k = i + 1; k <= N; ++k) Hn[k] = fma_t(Hn[k], zc * rk[k - i + 1], a);
    }
    if constexpr (U >= 1) {
        if constexpr (U == 1) {
#pragma unroll
            for (int c = 0; c < D; ++c) B1[c] = fma_t(Hn[P + 1], zu[c], B1[c]);
        } else {
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const T t1 = fma_t(Hn[P + 2], zu[c] * rk[2], B1[c]);   // T^(N)_{P+1}[u c]
                B1[c] = fma_t(Hn[P + 1], zu[c], B1[c]);
#pragma unroll
                for (int j = 0; j < D; ++j) B2[c * D + j] = fma_t(t1, zu[j], B2[c * D + j]);
            }
        }
    }
}

// (A, B1, B2) <- (A, B1, B2) [x] C, as StretchFactor but for both levels below the word.
template <typename T, int D, int P, int U>
__device__ __forceinline__ void split_multiply(T *A, T *B1, T *B2, const uint32_t *pre, const T *C)
{
    if constexpr (U == 2) {
        T z[D], own[D * D];
#pragma unroll
        for (int c = 0; c < D * D; ++c) own[c] = C[stretch_off(D, P + 2) + pre[P] * (D * D) + c];
#pragma unroll
        for (int e = 0; e < D; ++e) z[e] = C[e];
#pragma unroll
        for (int c = 0; c < D; ++c)
#pragma unroll
            for (int e = 0; e < D; ++e) own[c * D + e] = fma_t(B1[c], z[e], own[c * D + e]);
#pragma unroll
        for (int j = 1; j <= P; ++j) {
            const T *r = j < P ? C + stretch_off(D, P - j + 2) + suffix_word<D>(pre, j, P) * (D * D) : C + stretch_off(D, 2);
#pragma unroll
            for (int c = 0; c < D * D; ++c) own[c] = fma_t(A[j], r[c], own[c]);
        }
#pragma unroll
        for (int c = 0; c < D * D; ++c) B2[c] += own[c];
    }
    StretchFactor<T, D, P> f;
    f.read(pre, C);
    f.multiply(A, B1);
}

// Rows (paths) in K = 2^log2K stretches of m increments, `paths` rows to a workgroup; dynamic LDS: the larger of the staged increments
// and half the stretches' signatures.
template <typename T, int D, int N>
__global__ void __launch_bounds__((SplitShape<T, D, N>::kThreads))
sig_tree_split_kernel(Shape sh, int log2K, int m, int paths, const T *__restrict__ path, T *__restrict__ out)
{
    using SS = SplitShape<T, D, N>;
    constexpr int U = SS::U, P = SS::P, W = SS::kWords;
    constexpr int64_t kS = tree_off(D, N + 1);
    extern __shared__ __align__(16) unsigned char split_smem[];
    T *lds = reinterpret_cast<T *>(split_smem);

    const int K = 1 << log2K, tid = threadIdx.x;
    const int stream_raw = tid / W, u = tid - stream_raw * W;   // which stretch of the workgroup's, which word
    const int streams = paths << log2K;
    const int stream = stream_raw < streams ? stream_raw : streams - 1;   // threads beyond the last idle along
    const int c = stream & (K - 1), slot = stream >> log2K;
    const int64_t row_raw = int64_t(blockIdx.x) * paths + slot, row = row_raw < sh.B ? row_raw : sh.B - 1;
    const bool live = stream_raw < streams && row_raw < sh.B;

    int cl[P + 1];
    uint32_t pre[P + 1] = {};
    {
        uint32_t rest = uint32_t(u);
#pragma unroll
        for (int i = P; i >= 1; --i) {
            pre[i] = rest;
            cl[i] = int(rest % D);
            rest /= D;
        }
    }
    T rk[N + 2];
#pragma unroll
    for (int k = 1; k <= N + 1; ++k) rk[k] = T(1) / T(k);
    T A[P + 1] = {}, B1[D] = {}, B2[U == 2 ? D * D : 1] = {};

    // the stretch's increments, staged by its own threads
    const int64_t inc0 = int64_t(c) * m;
    const int n = int(sh.n_inc - inc0 < 0 ? 0 : sh.n_inc - inc0 < m ? sh.n_inc - inc0 : m);
    const T *x = path + row * sh.L * D, *bpv = static_cast<const T *>(sh.basepoint_value);
    T hi[SS::kPerThread], lo[SS::kPerThread];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int q = 0; q < SS::kPerThread; ++q) {
            const int e = u + W * q < kSplitTile * D ? u + W * q : kSplitTile * D - 1, i = e / D, ch = e - i * D;
            const bool on = t0 + i < n;
            const int64_t i_hi = (on ? inc0 + t0 + i : 0) + (sh.basepoint ? 0 : 1);   // unconditional loads, inside the path
            const bool first = i_hi == 0;   // the increment from the basepoint
            hi[q] = x[i_hi * D + ch];
            lo[q] = bpv != nullptr && first ? bpv[row * D + ch] : x[(first ? 0 : i_hi - 1) * D + ch];
            if (first && bpv == nullptr) lo[q] = T(0);
            if (!on) lo[q] = hi[q];
        }
    };
    fetch(0);
    T *zrow0 = lds + stream * SS::kRow;
    for (int t0 = 0; t0 < m; t0 += kSplitTile) {
        __syncthreads();
        if (stream_raw < streams) {
#pragma unroll
            for (int q = 0; q < SS::kPerThread; ++q)
                if (u + W * q < kSplitTile * D) zrow0[u + W * q] = hi[q] - lo[q];
        }
        __syncthreads();
        if (t0 + kSplitTile < m) fetch(t0 + kSplitTile);
        const int nt = n - t0 < kSplitTile ? n - t0 : kSplitTile;   // its own: a zero increment is not nothing beside an infinity
        const T *zrow = zrow0;
        for (int s = 0; s < nt; ++s, zrow += D) split_increment<T, D, N, U>(zrow, cl, rk, A, B1, B2);
    }

    auto store = [&](T *o) {   // a prefix is written by the first thread below it
        uint32_t width = 1;
#pragma unroll
        for (int i = P; i >= 1; --i) {
            if (uint32_t(u) % width == 0) o[tree_off(D, i) + pre[i]] = A[i];
            width *= D;
        }
#pragma unroll
        for (int ch = 0; ch < D; ++ch) o[tree_off(D, P + 1) + u * D + ch] = B1[ch];
        if constexpr (U == 2) {
#pragma unroll
            for (int ch = 0; ch < D * D; ++ch) o[tree_off(D, P + 2) + u * (D * D) + ch] = B2[ch];
        }
    };
    for (int r = 0; r < log2K; ++r) {   // neighbours of 2^r stretches joined
        const int half = 1 << r;
        T *right = lds + ((slot << (log2K - 1 - r)) + (c >> (r + 1))) * kS;
        __syncthreads();   // what the LDS held has been read
        if (live && (c & (2 * half - 1)) == half) store(right);
        __syncthreads();
        if (live && (c & (2 * half - 1)) == 0 && inc0 + int64_t(half) * m < sh.n_inc) split_multiply<T, D, P, U>(A, B1, B2, pre, right);
    }
    if (live && c == 0) store(out + row * kS);
}

// Stretches (a power of two, up to 256 in fp32 and 128 in fp64 at d = 2; 1: none) for a batch: as many as a workgroup holds, of 8 increments
// and more, while the threads before the last doubling are one wavefront per SIMD or less (100 points, in one piece | cut: 500 x d = 5, N = 5,
// 62 500 threads 23.8 | 15.2 us; 1040 x d = 3, N = 5 18.4 | 9.6; 2306 x 667, d = 2, N = 6, fp64 197 | 81; in fp64 from six channels on, where a
// workgroup has a compute unit to itself, up to 24 000: 286 x 162, d = 6, N = 5, 62 000 threads 65 | 73).  Below 32 increments there is nothing to
// gain (9 us either way), nor below 64 from two stretches (1 x 51, d = 4, N = 6, fp64 12.2 | 13.0), below 40 at d = 6, N = 5, where 37 KB a
// signature are to be joined (102 x 33 10.7 | 12.3; 7 x 45 even), or below 128 at d = 8, N = 4 in fp64, where a thread's share spills (16 x 97
// 1.14 times one piece, 130 0.94, 260 0.61).
template <typename T, int D, int N>
int split_count(const Shape &sh)
{
    using SS = SplitShape<T, D, N>;
    constexpr int64_t kS = tree_off(D, N + 1), kFull = sizeof(T) == 8 && D >= 6 ? 24000 : 64 * 1024;
    constexpr bool kSpills = sizeof(T) == 8 && D == 8 && SS::U == 2;
    constexpr int64_t kShortest = kSpills ? 128 : 4 * SS::kAllWords > SS::kThreads ? 64 : kS * int64_t(sizeof(T)) > 32 * 1024 ? 40 : 32;
    if (sh.n_inc < kShortest || sh.n_inc > (int64_t(1) << 30)) return 1;
    int K = 1;
    while (2 * K * SS::kAllWords <= SS::kThreads && sh.n_inc >= 16 * K && int64_t(K) * kS * int64_t(sizeof(T)) <= kSplitLds &&
           sh.B <= kFull / (K * SS::kWords))
        K *= 2;
    return K;
}

template <typename T, int D, int N>
hipError_t launch_split_dn(const Shape &sh, const T *path, T *out, hipStream_t st, int *count)
{
    using SS = SplitShape<T, D, N>;
    constexpr int64_t kS = tree_off(D, N + 1);
    const int K = split_count<T, D, N>(sh);
    if (count != nullptr) *count = K;
    if (K == 1 || count != nullptr) return hipErrorNotSupported;
    int log2K = 0;
    while (1 << log2K < K) ++log2K;
    int64_t paths = 256 / (K * SS::kWords);   // whole paths to a workgroup of four wavefronts
    const int64_t fit = kSplitLds / (K / 2 * kS * int64_t(sizeof(T)));
    paths = paths < 1 ? 1 : paths > fit ? fit : paths;
    const int m = int((sh.n_inc + K - 1) / K), threads = int(paths * K * SS::kWords + 63) / 64 * 64;
    const int64_t staged = paths * K * SS::kRow, joined = paths * (K / 2) * kS, groups = (sh.B + paths - 1) / paths;
    const size_t lds = size_t(staged > joined ? staged : joined) * sizeof(T);
    if (groups > 0x3fffff || lds > size_t(kSplitLds)) return hipErrorNotSupported;
    if (lds > 64 * 1024) {   // the most of any call: the attribute is the process's, another thread may set it in between
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(sig_tree_split_kernel<T, D, N>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kSplitLds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((sig_tree_split_kernel<T, D, N>), dim3(unsigned(groups)), dim3(unsigned(threads)), lds, st, sh, log2K, m, int(paths),
                       path, out);
    return hipGetLastError();
}

template <typename T, int D, int N>
hipError_t launch_split_n(const Shape &sh, const T *path, T *out, hipStream_t st, int *count)
{
    if constexpr (2 * SplitShape<T, D, N>::kAllWords <= SplitShape<T, D, N>::kThreads && tree_off(D, N + 1) * int64_t(sizeof(T)) <= kSplitLds)
        return launch_split_dn<T, D, N>(sh, path, out, st, count);
    else
        return hipErrorNotSupported;
}

// hipErrorNotSupported, with nothing enqueued, where the batch fills the chip or a path the workgroup; `count`, if given, takes the number
// of stretches instead.
template <typename T, int D>
hipError_t launch_split_d(const Shape &sh, const T *path, T *out, hipStream_t st, int *count)
{
    switch (sh.N) {
        case 3: return launch_split_n<T, D, 3>(sh, path, out, st, count);
        case 4: return launch_split_n<T, D, 4>(sh, path, out, st, count);
        case 5: return launch_split_n<T, D, 5>(sh, path, out, st, count);
        case 6: return launch_split_n<T, D, 6>(sh, path, out, st, count);
    }
    if constexpr (D <= 8) {
        switch (sh.N) {
            case 7: return launch_split_n<T, D, 7>(sh, path, out, st, count);
            case 8: return launch_split_n<T, D, 8>(sh, path, out, st, count);
            case 9: return launch_split_n<T, D, 9>(sh, path, out, st, count);
        }
    }
    return hipErrorNotSupported;
}

}  // namespace
}  // namespace sig

#endif  // SIG_TREE_SPLIT_IMPL_H_
