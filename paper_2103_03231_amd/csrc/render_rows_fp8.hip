// render_rows_fp8.hip - render kernels with fp8 networks and tiles of 32 or 64
// rays, for calls that do not fill the chip with the main kernel's tiles; top-N
// and inverse-CDF placement, both depth-network inputs.
#include "rows_kernel.h"

namespace donerf {

hipError_t launch_rows_fp8(int cdf, int ncap, int din, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    return a.tile_rays == 32   ? launch_rows<kFP8, 1>(cdf, ncap, din, a, grid, stream)
           : a.tile_rays == 64 ? launch_rows<kFP8, 2>(cdf, ncap, din, a, grid, stream)
                               : hipErrorInvalidValue;   // no such tile
}

}  // namespace donerf
