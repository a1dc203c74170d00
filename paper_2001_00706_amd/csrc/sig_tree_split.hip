// Prefix-tree scan of few paths with several stretches of a path to a workgroup (see sig_tree_split_impl.h).
#include "sig_tree_split_impl.h"

namespace sig {

template <typename T>
hipError_t launch_tree_split_t(const Shape &sh, const T *path, T *out, hipStream_t st, int *count = nullptr)
{
    if (sh.stream || sh.chunks > 1 || !tree_supported(sh)) return hipErrorNotSupported;
    switch (sh.d) {
        case 2: return launch_split_d<T, 2>(sh, path, out, st, count);
        case 3: return launch_split_d<T, 3>(sh, path, out, st, count);
        case 4: return launch_split_d<T, 4>(sh, path, out, st, count);
        case 5: return launch_split_d<T, 5>(sh, path, out, st, count);
        case 6: return launch_split_d<T, 6>(sh, path, out, st, count);
        case 7: return launch_split_d<T, 7>(sh, path, out, st, count);
        case 8: return launch_split_d<T, 8>(sh, path, out, st, count);
        case 9: return launch_split_d<T, 9>(sh, path, out, st, count);
        case 10: return launch_split_d<T, 10>(sh, path, out, st, count);
        case 11: return launch_split_d<T, 11>(sh, path, out, st, count);
        case 12: return launch_split_d<T, 12>(sh, path, out, st, count);
        case 13: return launch_split_d<T, 13>(sh, path, out, st, count);
        case 14: return launch_split_d<T, 14>(sh, path, out, st, count);
        case 15: return launch_split_d<T, 15>(sh, path, out, st, count);
        case 16: return launch_split_d<T, 16>(sh, path, out, st, count);
    }
    return hipErrorNotSupported;
}

hipError_t launch_tree_split_f32(const Shape &sh, const float *path, float *out, hipStream_t st) { return launch_tree_split_t(sh, path, out, st); }
hipError_t launch_tree_split_f64(const Shape &sh, const double *path, double *out, hipStream_t st) { return launch_tree_split_t(sh, path, out, st); }


int tree_split_stretches(const Shape &sh, sig_dtype dtype)
{
    int count = 1;
    if (dtype == SIG_F32)
        launch_tree_split_t<float>(sh, nullptr, nullptr, nullptr, &count);
    else
        launch_tree_split_t<double>(sh, nullptr, nullptr, nullptr, &count);
    return count;
}

}  // namespace sig
