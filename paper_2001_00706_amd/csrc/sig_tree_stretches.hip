// fp32 instantiation of the prefix-tree gradient kernels for stretches of paths (see sig_tree_backward_impl.h).
#include "sig_tree_backward_impl.h"

namespace sig {

bool tree_stretches_supported(const Shape &sh) { return !sh.stream && sh.d >= 2 && sh.d <= 8 && sh.N >= 3 && sh.N <= kTbMaxDepth && tb_workspace_bytes(sh, 4) >= 0; }

// Nodes of all levels above K stretches, where they are formed from the fewest stretches on (8: launch_tb_stretches_dn).
int64_t tree_stretch_nodes(int64_t K)
{
    int64_t nodes = 0;
    for (int64_t n = K; n > 8; nodes += n) n = (n + (1 << kStretchRadixLog2) - 1) >> kStretchRadixLog2;
    return nodes;
}

hipError_t launch_tree_stretches_f32(const Shape &sh, int64_t K, int64_t m, const float *path, const float *C, float *group, const float *gout,
                                     float *gpath, float *gbase, void *partial, hipStream_t st)
{
    return launch_tb_stretches<float>(sh, K, m, path, C, group, gout, gpath, gbase, static_cast<float *>(partial), st);
}

}  // namespace sig
