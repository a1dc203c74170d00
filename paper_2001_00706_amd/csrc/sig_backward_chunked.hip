// Pieces of the gradient of few long paths, the scan cut into stretches (final mode; paper sections 5.1 and 5.3).
//
// The gradient by reversibility (appendix C.1) walks a path backwards an increment at a time, so one path keeps one
// workgroup busy for its whole length.  Cut into K stretches of m increments, with C_c the signature of stretch c alone
// and S_c = C_0 [x] .. [x] C_c that of the path up to the end of stretch c (Chen's identity, section 2.2), the walk
// over stretch c needs two things at its end: S_c, and the gradient g_c of the loss with respect to S_c.  The first is
// a running product.  The second follows from S_c = S_{c-1} [x] C_c, which is linear in S_{c-1}:
//     g_{c-1}[u] = sum_v g_c[u v] C_c[v],      v over all words with |u v| <= N, the empty one (C[empty] = 1) included,
// starting from g_{K-1} = the gradient with respect to the whole signature.  Given both, the stretches are independent
// and the ordinary gradient kernels serve them as B K short paths.
// One stretch after the other, both recurrences would be chains of K steps of a few microseconds each.  The product is
// associative, so the S_c and the products T_c = C_{c+1} [x] .. [x] C_{K-1} of what comes after a stretch are formed along a
// binary tree in 2 log2 K rounds (sig_product_tree.hip), and every g_c comes from the last one in one step,
//     g_c[u] = sum_v g_{K-1}[u v] T_c[v].
// With so many paths that one product of all of them fills the chip, the chains take a third of the products and are used
// (products_in_chains in sig_api.hip).
// For 2 to 8 channels at depths 3 to 9 the walk itself forms what a stretch needs and this file is not used
// (launch_tb_stretches in sig_tree_backward_impl.h).
// This file holds the plumbing around the gradient kernels: copying the stretches out as paths of their own (m + 1 points, the
// last point of a path repeated where the last stretch is short: increments of zero change no signature), the step from
// g_{K-1} to every g_c, and adding the stretches' point gradients up (a point shared by two stretches ends an increment of
// one and starts one of the other; the repeated last points sum to the gradient of the increment that ends at the real one).
#include "sig_internal.h"
#include "sig_lane_ops.h"

namespace sig {
namespace {

template <typename T>
__global__ void __launch_bounds__(256)
sig_stretch_gather_kernel(Shape sh, int64_t K, int64_t m, const T *__restrict__ path, T *__restrict__ rows)
{
    const int d = sh.d;
    const int64_t per_row = (m + 1) * d, total = sh.B * K * per_row;
    const T *bpv = static_cast<const T *>(sh.basepoint_value);
    for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < total; e += int64_t(gridDim.x) * 256) {
        const int64_t r = e / per_row, rest = e - r * per_row;
        const int64_t i = rest / d;
        const int ch = int(rest - i * d);
        const int64_t b = r / K, c = r - b * K;
        int64_t k = c * m + i;   // number of the point inside the scan, 0 .. n_inc
        if (k > sh.n_inc) k = sh.n_inc;
        T v;
        if (sh.basepoint)
            v = k == 0 ? (bpv != nullptr ? bpv[b * d + ch] : T(0)) : path[(b * sh.L + k - 1) * d + ch];
        else
            v = path[(b * sh.L + k) * d + ch];
        rows[e] = v;
    }
}

// How the words of each level are spread over a wavefront's lanes: a word of level i sums sum_{j = 1 .. N - i} d^j products,
// and teams of 2^team_log2[i] lanes (1, 4, 16 or 64) share a word's sums.
struct AdjointTeams {
    unsigned char team_log2[SIG_MAX_DEPTH + 1];
};

struct AdjointLevels {
    int words[SIG_MAX_DEPTH + 2];   // d^i
    int off[SIG_MAX_DEPTH + 2];     // offset of level i; off[N + 1] = S
    int team_log2[SIG_MAX_DEPTH + 2];
};

// The level tables as 32-bit numbers in LDS (S < 2^31), written by one thread at positions known at compile time: the
// shape sits in scalar registers, where a run-time index would move it to scratch memory.  Needs a barrier after it.
__device__ __forceinline__ void adjoint_levels_fill(const Shape &sh, const AdjointTeams &teams, AdjointLevels *lv)
{
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k <= SIG_MAX_DEPTH; ++k) {
            lv->words[k] = int(sh.pw[k]);
            lv->off[k] = int(sh.off[k]);
            lv->team_log2[k] = teams.team_log2[k];
        }
        lv->off[SIG_MAX_DEPTH + 1] = int(sh.off[SIG_MAX_DEPTH + 1]);
    }
}

// gout = the gradient gin carried through the right multiplication by the signature cs.  For a word u of level i the
// sum over the words v of level j is a dot product of d^j consecutive scalars of level i + j of gin with level j of cs.
// An item is a wavefront's worth of teams of one level; the calling wavefront takes the items item0, item0 + step, .. of
// every level (STEP > 0: step is that constant, and the levels' items are dealt out in turn so that no wavefront is
// always first).  The order of the additions is fixed.
template <typename T, int STEP>
__device__ __forceinline__ void stretch_adjoint_items(int N, int d, const AdjointLevels *lv, const T *gin, const T *cs, T *gout,
                                                      int item0, int step_runtime)
{
    const int lane = threadIdx.x & 63;
    const int step = STEP > 0 ? STEP : step_runtime;
    int dealt = 0;
    for (int i = 1; i <= N; ++i) {
        const int words = lv->words[i], base = lv->off[i], after = lv->off[i + 1];
        const int log2 = lv->team_log2[i], team = 1 << log2, per_item = 64 >> log2;
        const int items = (words + per_item - 1) >> (6 - log2);
        const int member = lane & (team - 1);
        const int first = STEP > 0 ? ((item0 - dealt) & (STEP - 1)) : item0;
        for (int t = first; t < items; t += step) {
            const int word = t * per_item + (lane >> log2);
            const bool on = word < words;
            T acc = T(0);
            if (on) {
                int pwj = 1, offj = 0, offn = after;   // d^j, the offset of level j, the offset of level i + j
                for (int j = 1; j <= N - i; ++j) {
                    pwj *= d;
                    const T *seg = gin + offn + word * pwj, *cj = cs + offj;
#pragma unroll 4
                    for (int v = member; v < pwj; v += team) acc += seg[v] * cj[v];
                    offj += pwj;
                    offn += words * pwj;
                }
            }
            for (int hop = team >> 1; hop >= 1; hop >>= 1) acc += __shfl_xor(acc, hop, 64);   // the same for every lane
            if (on && member == 0) gout[base + word] = acc + gin[base + word];
        }
        if (STEP > 0) dealt = (dealt + items) & (STEP - 1);
    }
}

// g[b][c] = the gradient g_last[b] carried through the right multiplication by F[b][c]; the last stretch has nothing
// after it and takes g_last as it is.  A workgroup of WAVES wavefronts per stretch holds g_last and the levels of F that
// take part (below N: `used` scalars) in LDS.
template <typename T, int WAVES>
__global__ void __launch_bounds__(64 * WAVES)
sig_stretch_adjoint_all_kernel(Shape sh, AdjointTeams teams, int64_t K, int used, const T *__restrict__ F, const T *__restrict__ g_last,
                               T *__restrict__ g)
{
    extern __shared__ __align__(16) unsigned char adjoint_smem[];
    __shared__ AdjointLevels lv;
    const int S = int(sh.S), tid = threadIdx.x;
    const int64_t r = blockIdx.x, b = r / K;
    T *gl = reinterpret_cast<T *>(adjoint_smem), *fl = gl + S;
    const T *g_row = g_last + b * sh.S, *f_row = F + r * sh.S;
    T *out = g + r * sh.S;
    if (r - b * K == K - 1) {
        for (int e = tid; e < S; e += 64 * WAVES) out[e] = g_row[e];
        return;
    }
    adjoint_levels_fill(sh, teams, &lv);
    for (int e = tid; e < S; e += 64 * WAVES) gl[e] = g_row[e];
    for (int e = tid; e < used; e += 64 * WAVES) fl[e] = f_row[e];
    __syncthreads();
    stretch_adjoint_items<T, WAVES>(sh.N, sh.d, &lv, gl, fl, out, tid >> 6, WAVES);
}

// The same straight from memory, for signatures that do not fit the LDS: the items of a stretch are spread over the grid.
template <typename T>
__global__ void __launch_bounds__(256)
sig_stretch_adjoint_each_kernel(Shape sh, AdjointTeams teams, int64_t rows, int64_t K, const T *__restrict__ F,
                                const T *__restrict__ g_last, T *__restrict__ g)
{
    __shared__ AdjointLevels lv;
    adjoint_levels_fill(sh, teams, &lv);
    __syncthreads();
    for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
        const int64_t b = r / K;
        const T *g_row = g_last + b * sh.S;
        T *out = g + r * sh.S;
        if (r - b * K == K - 1) {
            for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < sh.S; e += int64_t(gridDim.x) * 256) out[e] = g_row[e];
            continue;
        }
        stretch_adjoint_items<T, 0>(sh.N, sh.d, &lv, g_row, F + r * sh.S, out, int(blockIdx.x) * 4 + (threadIdx.x >> 6),
                                    int(gridDim.x) * 4);
    }
}

// One step of the chain: `out`, the gradient with respect to one of a path's K rows, from that with respect to the row after it and
// that row's own signature, a path per grid row.  The first step also copies the gradient it starts from into its row (`copy`).
template <typename T>
__global__ void __launch_bounds__(256)
sig_stretch_adjoint_step_kernel(Shape sh, AdjointTeams teams, int64_t stride, const T *from, int64_t from_stride, const T *__restrict__ C,
                                T *out, T *copy)
{
    __shared__ AdjointLevels lv;
    adjoint_levels_fill(sh, teams, &lv);
    __syncthreads();
    const int64_t b = blockIdx.y;
    if (copy != nullptr)
        for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < sh.S; e += int64_t(gridDim.x) * 256)
            copy[b * stride + e] = from[b * from_stride + e];
    stretch_adjoint_items<T, 0>(sh.N, sh.d, &lv, from + b * from_stride, C + b * stride, out + b * stride,
                                int(blockIdx.x) * 4 + (threadIdx.x >> 6), int(gridDim.x) * 4);
}

// Point gradients of the stretches [B K][m + 1][d] added up into those of the paths (and of the basepoints).
template <typename T>
__global__ void __launch_bounds__(256)
sig_stretch_scatter_kernel(Shape sh, int64_t K, int64_t m, const T *__restrict__ grows, T *__restrict__ gpath, T *__restrict__ gbase)
{
    const int d = sh.d;
    const int64_t n = sh.n_inc, per_path = (n + 1) * d, total = sh.B * per_path, per_row = (m + 1) * d;
    for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < total; e += int64_t(gridDim.x) * 256) {
        const int64_t b = e / per_path, rest = e - b * per_path;
        const int64_t k = rest / d;   // number of the point inside the scan
        const int ch = int(rest - k * d);
        const T *rows = grows + b * K * per_row;
        T sum;
        if (k < n) {
            const int64_t c = k / m, i = k - c * m;
            sum = rows[c * per_row + i * d + ch];
            if (i == 0 && c > 0) sum += rows[(c - 1) * per_row + m * d + ch];   // it also ends the stretch before
        } else {
            // the last point and its copies behind it in the last stretch
            const int64_t c = (n - 1) / m;
            sum = T(0);
            for (int64_t i = n - c * m; i <= m; ++i) sum += rows[c * per_row + i * d + ch];
        }
        if (sh.basepoint) {
            if (k == 0) {
                if (gbase != nullptr) gbase[b * d + ch] = sum;
            } else {
                gpath[(b * sh.L + k - 1) * d + ch] = sum;
            }
        } else {
            gpath[(b * sh.L + k) * d + ch] = sum;
        }
    }
}

unsigned grid_for(int64_t elems)
{
    const int64_t groups = (elems + 255) / 256;
    return unsigned(groups < 1 ? 1 : groups < 65536 ? groups : 65536);
}

template <typename T>
hipError_t stretch_gather(const Shape &sh, int64_t K, int64_t m, const T *path, T *rows, hipStream_t st)
{
    hipLaunchKernelGGL((sig_stretch_gather_kernel<T>), dim3(grid_for(sh.B * K * (m + 1) * sh.d)), dim3(256), 0, st, sh, K, m, path, rows);
    return hipGetLastError();
}

// The teams of every level, and how many items they make in all.
AdjointTeams adjoint_teams(const Shape &sh, int64_t &items)
{
    AdjointTeams teams;
    items = 0;
    for (int i = 0; i <= SIG_MAX_DEPTH; ++i) teams.team_log2[i] = 0;
    for (int i = 1; i <= sh.N; ++i) {
        int64_t cost = 0;
        for (int j = 1; i + j <= sh.N; ++j) cost += sh.pw[j];
        teams.team_log2[i] = cost <= 8 ? 0 : cost <= 64 ? 2 : cost <= 512 ? 4 : 6;
        const int64_t per_item = 64 >> teams.team_log2[i];
        items += (sh.pw[i] + per_item - 1) / per_item;
    }
    return teams;
}

size_t adjoint_lds(const Shape &sh, size_t elem) { return (size_t(sh.S) + size_t(sh.off[sh.N])) * elem; }   // g_last, levels of F below N

bool adjoint_in_lds(const Shape &sh, size_t elem) { return adjoint_lds(sh, elem) + sizeof(AdjointLevels) <= 64 * 1024; }

template <typename T>
hipError_t stretch_adjoint_all(const Shape &sh, int64_t K, const T *F, const T *g_last, T *g, hipStream_t st)
{
    int64_t items = 0;
    const AdjointTeams teams = adjoint_teams(sh, items);
    const int64_t used = sh.off[sh.N];
    const size_t lds = adjoint_lds(sh, sizeof(T));
    if (adjoint_in_lds(sh, sizeof(T)) && sh.B <= 0xffffffffll / 1024) {   // a grid has less than 2^32 threads
        if (sh.S >= 1024)
            hipLaunchKernelGGL((sig_stretch_adjoint_all_kernel<T, 16>), dim3(unsigned(sh.B)), dim3(1024), lds, st, sh, teams, K, int(used),
                               F, g_last, g);
        else
            hipLaunchKernelGGL((sig_stretch_adjoint_all_kernel<T, 4>), dim3(unsigned(sh.B)), dim3(256), lds, st, sh, teams, K, int(used), F,
                               g_last, g);
        return hipGetLastError();
    }
    const int64_t groups = (items + 3) / 4;
    const dim3 grid(unsigned(groups < 4096 ? groups : 4096), unsigned(sh.B < 65535 ? sh.B : 65535));
    hipLaunchKernelGGL((sig_stretch_adjoint_each_kernel<T>), grid, dim3(256), 0, st, sh, teams, sh.B, K, F, g_last, g);
    return hipGetLastError();
}

template <typename T>
hipError_t stretch_adjoint_chain(const Shape &sh, int64_t K, const T *C, const T *g_last, T *g, hipStream_t st)
{
    int64_t items = 0;
    const AdjointTeams teams = adjoint_teams(sh, items);
    const int64_t paths = sh.B / K, groups = (items + 3) / 4, stride = K * sh.S;   // sh.B counts stretches; at most 65535 paths
    const dim3 grid(unsigned(groups < 4096 ? groups : 4096), unsigned(paths));
    for (int64_t c = K - 1; c >= 1; --c) {
        const bool first = c == K - 1;
        T *row = g + c * sh.S;
        hipLaunchKernelGGL((sig_stretch_adjoint_step_kernel<T>), grid, dim3(256), 0, st, sh, teams, stride, first ? g_last : row,
                           first ? int64_t(sh.S) : stride, C + c * sh.S, row - sh.S, first ? row : nullptr);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

template <typename T>
hipError_t stretch_scatter(const Shape &sh, int64_t K, int64_t m, const T *grows, T *gpath, T *gbase, hipStream_t st)
{
    hipLaunchKernelGGL((sig_stretch_scatter_kernel<T>), dim3(grid_for(sh.B * (sh.n_inc + 1) * sh.d)), dim3(256), 0, st, sh, K, m, grows,
                       gpath, gbase);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_stretch_gather(const Shape &sh, sig_dtype dtype, int64_t K, int64_t m, const void *path, void *rows, hipStream_t st)
{
    return dtype == SIG_F32 ? stretch_gather(sh, K, m, static_cast<const float *>(path), static_cast<float *>(rows), st)
                            : stretch_gather(sh, K, m, static_cast<const double *>(path), static_cast<double *>(rows), st);
}

bool stretch_adjoint_in_lds(const Shape &sh, sig_dtype dtype) { return adjoint_in_lds(sh, dtype == SIG_F32 ? sizeof(float) : sizeof(double)); }

hipError_t launch_stretch_adjoint_all(const Shape &sh, sig_dtype dtype, int64_t K, const void *F, const void *g_last, void *g,
                                      hipStream_t st)
{
    return dtype == SIG_F32 ? stretch_adjoint_all(sh, K, static_cast<const float *>(F), static_cast<const float *>(g_last),
                                                  static_cast<float *>(g), st)
                            : stretch_adjoint_all(sh, K, static_cast<const double *>(F), static_cast<const double *>(g_last),
                                                  static_cast<double *>(g), st);
}

hipError_t launch_stretch_adjoint_chain(const Shape &sh, sig_dtype dtype, int64_t K, const void *C, const void *g_last, void *g,
                                        hipStream_t st)
{
    return dtype == SIG_F32 ? stretch_adjoint_chain(sh, K, static_cast<const float *>(C), static_cast<const float *>(g_last),
                                                    static_cast<float *>(g), st)
                            : stretch_adjoint_chain(sh, K, static_cast<const double *>(C), static_cast<const double *>(g_last),
                                                    static_cast<double *>(g), st);
}

hipError_t launch_stretch_scatter(const Shape &sh, sig_dtype dtype, int64_t K, int64_t m, const void *grows, void *gpath, void *gbase,
                                  hipStream_t st)
{
    return dtype == SIG_F32
               ? stretch_scatter(sh, K, m, static_cast<const float *>(grows), static_cast<float *>(gpath), static_cast<float *>(gbase), st)
               : stretch_scatter(sh, K, m, static_cast<const double *>(grows), static_cast<double *>(gpath), static_cast<double *>(gbase),
                                 st);
}

}  // namespace sig
