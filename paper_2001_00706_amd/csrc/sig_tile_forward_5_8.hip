// The tile kernels of 5 to 8 channels in final mode (see sig_tile_forward_impl.h).
#include "sig_tile_forward_impl.h"

namespace sig {

template hipError_t launch_tile_forward_d<5>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<6>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<7>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<8>(const Shape &, const float *, float *, hipStream_t);

}  // namespace sig
