// fp32 instantiation of the prefix-tree gradient kernels for stretches of paths in stream mode (see sig_tree_backward_impl.h).
#include "sig_tree_backward_impl.h"

namespace sig {

int64_t tree_stream_carried(const Shape &sh) { return sh.pw[sh.N - 2] * (sh.N - 2 + sh.d + int64_t(sh.d) * sh.d); }

hipError_t launch_tree_stream_stretches_f32(const Shape &sh, int64_t K, int64_t m, const float *path, const float *sig, const float *gout,
                                            const float *C, float *carried, float *gpath, float *gbase, void *partial, hipStream_t st)
{
    return launch_tb_stream_stretches<float>(sh, K, m, path, sig, gout, C, carried, gpath, gbase, static_cast<float *>(partial), st);
}

}  // namespace sig
