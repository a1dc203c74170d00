// fp64 instantiation of the prefix-tree gradient kernels for stretches of paths (see sig_tree_backward_impl.h).
#include "sig_tree_backward_impl.h"

namespace sig {

hipError_t launch_tree_stretches_f64(const Shape &sh, int64_t K, int64_t m, const double *path, const double *C, double *group, const double *gout,
                                     double *gpath, double *gbase, void *partial, hipStream_t st)
{
    return launch_tb_stretches<double>(sh, K, m, path, C, group, gout, gpath, gbase, static_cast<double *>(partial), st);
}

}  // namespace sig
