// fp64 instantiation of the prefix-tree gradient kernels for stretches of paths in stream mode (see sig_tree_backward_impl.h).
#include "sig_tree_backward_impl.h"

namespace sig {

hipError_t launch_tree_stream_stretches_f64(const Shape &sh, int64_t K, int64_t m, const double *path, const double *sig, const double *gout,
                                            const double *C, double *carried, double *gpath, double *gbase, void *partial, hipStream_t st)
{
    return launch_tb_stream_stretches<double>(sh, K, m, path, sig, gout, C, carried, gpath, gbase, static_cast<double *>(partial), st);
}

}  // namespace sig
