// Products of many signatures per path along a binary tree: the signatures of consecutive stretches of a path joined (Chen's
// identity, paper section 2.2, eq. "grouplike"; the reduction of section 5.1).
//
// Node i of level l stands for the stretches i 2^l .. min((i + 1) 2^l, K) - 1; level 0 is the stretches themselves.  Going
// up, P_{l+1}[i] = P_l[2i] [x] P_l[2i+1] (a last node without a neighbour moves up as it is); the node at the top is the
// whole path.  Where every prefix and every suffix is wanted, going down a node gets the product of everything up to and
// including it, I, and of everything after it, F:
//     I_l[2i+1] = I_{l+1}[i],   I_l[2i] = I_{l+1}[i-1] [x] P_l[2i],     F_l[2i+1] = F_{l+1}[i],   F_l[2i] = P_l[2i+1] [x] F_{l+1}[i].
// Both are kept in the row of the node's last stretch, where the right child's entry is its parent's, so a round
// writes the left children only and the rounds need one buffer each; the rows end up as the prefix signatures and the
// signatures of what comes after.  The inner nodes P_l need no buffer of their own: they lie in rows of I and F that are written
// in a later round than the last one that reads the node (tree_node).
//
// Where the paths alone fill the chip (the caller's rule says where), the prefixes are formed one after the other instead: a third
// of the products.
//
// A round is a launch over all words of all its products, which takes 4 to 6 us whatever its size: it is bound by the launch
// and one trip to memory.  The rounds near the top have little to do, so from the first level whose nodes hold at most
// kTopWords scalars per path on, one workgroup per path does all rounds up (and down) in a single launch, about 1.5 us a
// round (launches of their own beyond that: a workgroup would take longer than the launch it saves).
#include "sig_internal.h"
#include "sig_product.h"

namespace sig {
namespace {

constexpr int64_t kTopWords = 8192;
constexpr int kTopThreads = 1024;

// The K signatures of every path and the two results, [paths][K][S] each; `top` is the level of the single node.
template <typename T>
struct ScanRows {
    const T *C;
    T *I, *F;
    int64_t K;
    int top;
};

__host__ __device__ inline int64_t tree_nodes(int64_t K, int level) { return (K + (int64_t(1) << level) - 1) >> level; }

// The row of the last stretch of node i of level l.
__device__ __forceinline__ int64_t tree_slot(int64_t i, int level, int64_t K)
{
    const int64_t end = (i + 1) << level;
    return (end < K ? end : K) - 1;
}

// Where node i of level l of path b lies.  The top is the whole path, the last row of I.  Level 1 fills the even rows of I,
// which the last round writes (its last node goes to the spare last row of F where it would meet the top).  The levels
// above it follow one another (`before`: nodes of level 2 .. l - 1) in those rows of F that the last two rounds write, three
// of every four.
template <typename T>
__device__ __forceinline__ T *tree_node(const ScanRows<T> &r, int64_t S, int64_t b, int level, int64_t before, int64_t i)
{
    const int64_t row0 = b * r.K;
    if (level == 0) return const_cast<T *>(r.C) + (row0 + i) * S;
    if (level == r.top) return r.I + (row0 + r.K - 1) * S;
    if (level == 1) return 2 * i == r.K - 1 ? r.F + (row0 + r.K - 1) * S : r.I + (row0 + 2 * i) * S;
    const uint32_t x = uint32_t(before + i);
    return r.F + (row0 + int64_t(x + x / 3)) * S;
}

// The words at position p of out = a [x] b; a null factor is the identity.
template <typename T, typename V, int D>
__device__ __forceinline__ void tree_word(const Shape &sh, const T *a, const T *b, T *out, uint32_t p)
{
    *reinterpret_cast<V *>(out + p) = a == nullptr   ? *reinterpret_cast<const V *>(b + p)
                                      : b == nullptr ? *reinterpret_cast<const V *>(a + p)
                                                     : product_word<T, V, D>(a, b, p, uint32_t(sh.d));
}

// The factors of one product and where it goes.
template <typename T>
struct TreeProduct {
    const T *a, *b;
    T *out;
};

// Node i of level l + 1.  `before`: nodes of level 2 .. l - 1.
template <typename T>
__device__ __forceinline__ TreeProduct<T> tree_up(const ScanRows<T> &rows, int64_t S, int64_t b, int level, int64_t before, int64_t i)
{
    const int64_t n = tree_nodes(rows.K, level);
    return {tree_node(rows, S, b, level, before, 2 * i),
            2 * i + 1 < n ? tree_node(rows, S, b, level, before, 2 * i + 1) : nullptr,
            tree_node(rows, S, b, level + 1, level >= 2 ? before + n : 0, i)};
}

// Left child 2i of `level`: its I (which = 0) or F (which = 1).
template <typename T>
__device__ __forceinline__ TreeProduct<T> tree_down(const ScanRows<T> &rows, int64_t S, int64_t b, int level, int64_t before, int64_t i,
                                                    int which)
{
    const int64_t K = rows.K, to = tree_slot(2 * i, level, K) * S;
    T *I = rows.I + b * K * S, *F = rows.F + b * K * S;
    if (which == 0)
        return {i > 0 ? I + tree_slot(i - 1, level + 1, K) * S : nullptr, tree_node(rows, S, b, level, before, 2 * i), I + to};
    const int64_t end = tree_slot(i, level + 1, K);   // nothing comes after the last stretch
    return {tree_node(rows, S, b, level, before, 2 * i + 1), end < K - 1 ? F + end * S : nullptr, F + to};
}

// All words of a product by the workgroups of one grid row.
template <typename T, typename V, int D>
__device__ __forceinline__ void tree_row(const Shape &sh, const TreeProduct<T> &t)
{
    constexpr uint32_t kWords = sizeof(V) / sizeof(T);
    for (uint32_t v = blockIdx.x * 256 + threadIdx.x; v < uint32_t(sh.S) / kWords; v += gridDim.x * 256)
        tree_word<T, V, D>(sh, t.a, t.b, t.out, kWords * v);
}

// One round up: all nodes of level + 1.
template <typename T, typename V, int D>
__global__ void __launch_bounds__(256)
sig_tree_up_kernel(Shape sh, ScanRows<T> rows, int64_t paths, int level, int64_t before)
{
    const int64_t above = tree_nodes(rows.K, level + 1);
    for (int64_t r = blockIdx.y; r < paths * above; r += gridDim.y)
        tree_row<T, V, D>(sh, tree_up(rows, sh.S, r / above, level, before, r % above));
}

// One round down: the left children of `level`.  Every other row of the grid is a node's I, the ones between are the F.
template <typename T, typename V, int D>
__global__ void __launch_bounds__(256)
sig_tree_down_kernel(Shape sh, ScanRows<T> rows, int64_t paths, int level, int64_t before)
{
    const int64_t pairs = tree_nodes(rows.K, level) / 2;
    for (int64_t r = blockIdx.y; r < 2 * paths * pairs; r += gridDim.y)
        tree_row<T, V, D>(sh, tree_down(rows, sh.S, (r >> 1) / pairs, level, before, (r >> 1) % pairs, int(r & 1)));
}

// Every round from `level` on (at least two nodes, at most kTopWords scalars in all), up and down again, by one workgroup
// per path.
template <typename T, typename V, int D>
__global__ void __launch_bounds__(kTopThreads)
sig_tree_top_kernel(Shape sh, ScanRows<T> rows, int level, int64_t before)
{
    constexpr uint32_t kWords = sizeof(V) / sizeof(T);
    const uint32_t nv = uint32_t(sh.S) / kWords;
    const int64_t b = blockIdx.x;
    for (int l = level; l < rows.top; ++l) {
        const uint32_t total = uint32_t(tree_nodes(rows.K, l + 1)) * nv;
        for (uint32_t e = threadIdx.x; e < total; e += kTopThreads) {
            const uint32_t i = e / nv, v = e - i * nv;
            const TreeProduct<T> t = tree_up(rows, sh.S, b, l, before, i);
            tree_word<T, V, D>(sh, t.a, t.b, t.out, kWords * v);
        }
        if (l >= 2) before += tree_nodes(rows.K, l);
        __syncthreads();
    }
    for (int l = rows.top - 1; l >= level; --l) {
        if (l >= 2) before -= tree_nodes(rows.K, l);
        const uint32_t total = 2 * uint32_t(tree_nodes(rows.K, l) / 2) * nv;
        for (uint32_t e = threadIdx.x; e < total; e += kTopThreads) {
            const uint32_t r = e / nv, v = e - r * nv;
            const TreeProduct<T> t = tree_down(rows, sh.S, b, l, before, r >> 1, int(r & 1));
            tree_word<T, V, D>(sh, t.a, t.b, t.out, kWords * v);
        }
        __syncthreads();
    }
}

// Step c of the chain I_c = I_{c-1} [x] C_c; the first step also copies I_0 = C_0 (every other row of its grid).
template <typename T, typename V, int D>
__global__ void __launch_bounds__(256)
sig_chain_step_kernel(Shape sh, const T *__restrict__ C, T *I, int64_t paths, int64_t K, int64_t c)
{
    const int64_t each = c == 1 ? 2 : 1;
    for (int64_t r = blockIdx.y; r < each * paths; r += gridDim.y) {
        const int64_t row0 = r / each * K;
        if (r % each == 1) {
            tree_row<T, V, D>(sh, {C + row0 * sh.S, nullptr, I + row0 * sh.S});
        } else {
            const T *left = c == 1 ? C + row0 * sh.S : I + (row0 + c - 1) * sh.S;
            tree_row<T, V, D>(sh, {left, C + (row0 + c) * sh.S, I + (row0 + c) * sh.S});
        }
    }
}

// One round of the reduction: the n / 2 products of every path's n signatures P (n a power of two).
template <typename T, typename V, int D>
__global__ void __launch_bounds__(256)
sig_reduce_round_kernel(Shape sh, int64_t paths, int64_t n, const T *__restrict__ P, T *__restrict__ next)
{
    for (int64_t r = blockIdx.y; r < paths * (n / 2); r += gridDim.y) {
        const T *left = P + 2 * r * sh.S;
        tree_row<T, V, D>(sh, {left, left + sh.S, next + r * sh.S});
    }
}

// The rest of a reduction, from the n signatures P of every path (n >= 2, n S <= kTopWords) to their product; a path's own
// rows of P and its n / 2 rows of `spare` take turns as factors and results.
template <typename T, typename V, int D>
__global__ void __launch_bounds__(kTopThreads)
sig_reduce_top_kernel(Shape sh, int64_t n, T *P, T *spare, T *out)
{
    constexpr uint32_t kWords = sizeof(V) / sizeof(T);
    const uint32_t nv = uint32_t(sh.S) / kWords;
    const int64_t b = blockIdx.x;
    T *from = P + b * n * sh.S, *other = spare + b * (n / 2) * sh.S;
    for (int64_t count = n; count > 1;) {
        const int64_t above = count / 2;
        T *to = above > 1 ? other : out + b * sh.S;
        for (uint32_t e = threadIdx.x; e < uint32_t(above) * nv; e += kTopThreads) {
            const uint32_t i = e / nv, v = e - i * nv;
            const T *left = from + 2 * i * sh.S;
            tree_word<T, V, D>(sh, left, left + sh.S, to + i * sh.S, kWords * v);
        }
        __syncthreads();
        other = from;
        from = to;
        count = above;
    }
}

template <typename T, typename V, int D>
struct Tree {
    static constexpr int64_t kWords = sizeof(V) / sizeof(T);

    static dim3 grid(const Shape &sh, int64_t rows)
    {
        const int64_t groups = (sh.S / kWords + 255) / 256;
        return dim3(unsigned(groups < 4096 ? groups : 4096), unsigned(rows < 65535 ? rows : 65535));
    }

    // (a grid has less than 2^32 threads)
    static bool top_fits(const Shape &sh, int64_t paths, int64_t n) { return n * sh.S <= kTopWords && paths <= 0xffffffffll / kTopThreads; }

    static hipError_t scan(const Shape &sh, int64_t paths, int64_t K, const T *C, T *I, T *F, hipStream_t st)
    {
        ScanRows<T> rows = {C, I, F, K, 0};
        while (tree_nodes(K, rows.top) > 1) ++rows.top;
        int level = 0;
        int64_t before = 0;   // nodes of level 2 .. level - 1
        for (; level < rows.top && !top_fits(sh, paths, tree_nodes(K, level)); ++level) {
            hipLaunchKernelGGL((sig_tree_up_kernel<T, V, D>), grid(sh, paths * tree_nodes(K, level + 1)), dim3(256), 0, st, sh, rows, paths,
                               level, before);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
            if (level >= 2) before += tree_nodes(K, level);
        }
        if (level < rows.top) {
            hipLaunchKernelGGL((sig_tree_top_kernel<T, V, D>), dim3(unsigned(paths)), dim3(kTopThreads), 0, st, sh, rows, level, before);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        for (--level; level >= 0; --level) {
            if (level >= 2) before -= tree_nodes(K, level);
            hipLaunchKernelGGL((sig_tree_down_kernel<T, V, D>), grid(sh, 2 * paths * (tree_nodes(K, level) / 2)), dim3(256), 0, st, sh,
                               rows, paths, level, before);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    }

    static hipError_t chain(const Shape &sh, int64_t paths, int64_t K, const T *C, T *I, hipStream_t st)
    {
        for (int64_t c = 1; c < K; ++c) {
            hipLaunchKernelGGL((sig_chain_step_kernel<T, V, D>), grid(sh, c == 1 ? 2 * paths : paths), dim3(256), 0, st, sh, C, I, paths, K, c);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    }

    static hipError_t group(const Shape &sh, int64_t products, int R, const float *from, float *to, hipStream_t st)
    {
        return launch_reduce_group_f32(sh, products, R, from, to, st);
    }
    static hipError_t group(const Shape &sh, int64_t products, int R, const double *from, double *to, hipStream_t st)
    {
        return launch_reduce_group_f64(sh, products, R, from, to, st);
    }

    static hipError_t reduce(const Shape &sh, int64_t paths, int64_t K, T *C, T *spare, T *out, hipStream_t st)
    {
        T *from = C, *other = spare;
        int64_t n = K;
        // eight at a time: three rounds in the time of one and a half (400 shapes of up to 512 paths of 1024 chunks: 0.88 of a call's time, the worst
        // 23 paths of 2817 points, d = 5, N = 6, in 64 chunks 167 | 173 us)
        while (n > 1 && !top_fits(sh, paths, n)) {
            const int R = n >= 8 ? 8 : int(n);
            T *to = n > R ? other : out;
            const hipError_t err = group(sh, paths * (n / R), R, from, to, st);
            if (err == hipErrorNotSupported) break;
            if (err != hipSuccess) return err;
            other = from;
            from = to;
            n /= R;
        }
        while (n > 1 && !top_fits(sh, paths, n)) {
            const int64_t above = n / 2;
            T *to = above > 1 ? other : out;
            hipLaunchKernelGGL((sig_reduce_round_kernel<T, V, D>), grid(sh, paths * above), dim3(256), 0, st, sh, paths, n, from, to);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
            other = from;
            from = to;
            n = above;
        }
        if (n > 1) {
            hipLaunchKernelGGL((sig_reduce_top_kernel<T, V, D>), dim3(unsigned(paths)), dim3(kTopThreads), 0, st, sh, n, from, other,
                               out);
            return hipGetLastError();
        }
        return hipSuccess;
    }
};

template <typename T>
struct ScanCall {
    int64_t paths, K;
    const T *C;
    T *I, *F;

    uintptr_t addresses() const
    {
        return reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(I) | reinterpret_cast<uintptr_t>(F);
    }
    template <typename V, int D>
    hipError_t run(const Shape &sh, hipStream_t st) const { return Tree<T, V, D>::scan(sh, paths, K, C, I, F, st); }
};

template <typename T>
struct ChainCall {
    int64_t paths, K;
    const T *C;
    T *I;

    uintptr_t addresses() const { return reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(I); }
    template <typename V, int D>
    hipError_t run(const Shape &sh, hipStream_t st) const { return Tree<T, V, D>::chain(sh, paths, K, C, I, st); }
};

template <typename T>
struct ReduceCall {
    int64_t paths, K;
    T *C, *spare, *out;

    uintptr_t addresses() const
    {
        return reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(spare) | reinterpret_cast<uintptr_t>(out);
    }
    template <typename V, int D>
    hipError_t run(const Shape &sh, hipStream_t st) const { return Tree<T, V, D>::reduce(sh, paths, K, C, spare, out, st); }
};

template <typename T, typename Call>
hipError_t by_channels(const Shape &sh, const Call &call, hipStream_t st)
{
    typedef typename Four<T>::type V4;
    // four words at a time where the channel count and the buffers allow it (4 | d makes 4 | S)
    if (call.addresses() % (4 * sizeof(T)) == 0) {
        switch (sh.d) {
            case 4: return call.template run<V4, 4>(sh, st);
            case 8: return call.template run<V4, 8>(sh, st);
            case 12: return call.template run<V4, 12>(sh, st);
            case 16: return call.template run<V4, 16>(sh, st);
        }
    }
    switch (sh.d) {
        case 2: return call.template run<Siblings<T, 2>, 2>(sh, st);
        case 3: return call.template run<Siblings<T, 3>, 3>(sh, st);
        case 5: return call.template run<Siblings<T, 5>, 5>(sh, st);
        case 6: return call.template run<Siblings<T, 6>, 6>(sh, st);
        case 7: return call.template run<Siblings<T, 7>, 7>(sh, st);
    }
    return call.template run<T, 0>(sh, st);
}

}  // namespace

bool product_of_neighbours(int d) { return (d >= 2 && d <= 8) || d == 12 || d == 16; }

hipError_t launch_product_scan(const Shape &sh, sig_dtype dtype, int64_t paths, int64_t K, const void *C, void *I, void *F, hipStream_t st)
{
    if (dtype == SIG_F32)
        return by_channels<float>(sh, ScanCall<float>{paths, K, static_cast<const float *>(C), static_cast<float *>(I),
                                                      static_cast<float *>(F)}, st);
    return by_channels<double>(sh, ScanCall<double>{paths, K, static_cast<const double *>(C), static_cast<double *>(I),
                                                    static_cast<double *>(F)}, st);
}

hipError_t launch_product_chain(const Shape &sh, sig_dtype dtype, int64_t paths, int64_t K, const void *C, void *I, hipStream_t st)
{
    if (dtype == SIG_F32)
        return by_channels<float>(sh, ChainCall<float>{paths, K, static_cast<const float *>(C), static_cast<float *>(I)}, st);
    return by_channels<double>(sh, ChainCall<double>{paths, K, static_cast<const double *>(C), static_cast<double *>(I)}, st);
}

hipError_t launch_product_reduce(const Shape &sh, sig_dtype dtype, int64_t paths, int64_t K, void *C, void *spare, void *out,
                                 hipStream_t st)
{
    if (dtype == SIG_F32)
        return by_channels<float>(sh, ReduceCall<float>{paths, K, static_cast<float *>(C), static_cast<float *>(spare),
                                                        static_cast<float *>(out)}, st);
    return by_channels<double>(sh, ReduceCall<double>{paths, K, static_cast<double *>(C), static_cast<double *>(spare),
                                                      static_cast<double *>(out)}, st);
}

}  // namespace sig
