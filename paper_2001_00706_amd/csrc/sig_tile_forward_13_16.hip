// The tile kernels of 13 to 16 channels in final mode (see sig_tile_forward_impl.h).
#include "sig_tile_forward_impl.h"

namespace sig {

template hipError_t launch_tile_forward_d<13>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<14>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<15>(const Shape &, const float *, float *, hipStream_t);
template hipError_t launch_tile_forward_d<16>(const Shape &, const float *, float *, hipStream_t);

}  // namespace sig
