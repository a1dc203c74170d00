// The tile gradient kernels of 9 to 12 channels (see sig_tile_backward_impl.h).
#include "sig_tile_backward_impl.h"

namespace sig {

#define SIG_TILE(D)                                                                                                          \
    template hipError_t launch_tile_backward_d<D>(const Shape &, const float *, const float *, const float *, float *, float *, \
                                                  float *, hipStream_t);                                                     \
    template int tile_groups_d<D>(int64_t, int, int &);
SIG_TILE(9)
SIG_TILE(10)
SIG_TILE(11)
SIG_TILE(12)
#undef SIG_TILE

}  // namespace sig
