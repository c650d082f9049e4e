// render_rows_fp32.hip - render kernels with fp32 networks and tiles of 32
// rays, for calls that do not fill the chip with the main kernel's tiles; top-N
// and inverse-CDF placement, both depth-network inputs.
#include "rows_kernel.h"

namespace donerf {

hipError_t launch_rows_fp32(int cdf, int ncap, int din, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    if (a.tile_rays != 32) return hipErrorInvalidValue;   // no such tile
    return cdf ? launch_rows<kF32, 1, true>(ncap, din, a, grid, stream)
               : launch_rows<kF32, 1, false>(ncap, din, a, grid, stream);
}

}  // namespace donerf
