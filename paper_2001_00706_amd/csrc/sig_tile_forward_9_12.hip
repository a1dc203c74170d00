// The tile kernels of 9 to 12 channels in final mode (see sig_tile_forward_impl.h).
#include "sig_tile_forward_impl.h"

namespace sig {

template hipError_t launch_tile_forward_d<9>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<10>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<11>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<12>(const Shape &, const float *, float *, hipStream_t);

}  // namespace sig
