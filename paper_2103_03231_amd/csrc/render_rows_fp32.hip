// render_rows_fp32.hip - render kernels with fp32 networks: tiles of 64 rays, and
// of 32 for calls that do not fill the chip with those; top-N and inverse-CDF
// placement, both depth-network inputs.
#include "rows_kernel.h"

namespace donerf {

hipError_t launch_rows_fp32(int cdf, int ncap, int din, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    return a.tile_rays == 32             ? launch_rows<kF32, 1>(cdf, ncap, din, a, grid, stream)
           : a.tile_rays == 32 * kF32CB ? launch_rows<kF32, kF32CB>(cdf, ncap, din, a, grid, stream)
                                         : hipErrorInvalidValue;   // no such tile
}

}  // namespace donerf
