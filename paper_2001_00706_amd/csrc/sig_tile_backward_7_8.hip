// The tile gradient kernels of 7 to 8 channels (see sig_tile_backward_impl.h).
#include "sig_tile_backward_impl.h"

namespace sig {

#define SIG_TILE(D)                                                                                                          \
    template hipError_t launch_tile_backward_d<D>(const Shape &, const float *, const float *, const float *, float *, float *, \
                                                  float *, hipStream_t);                                                     \
    template int tile_groups_d<D>(int64_t, int, int &);
SIG_TILE(7)
SIG_TILE(8)
#undef SIG_TILE

}  // namespace sig
