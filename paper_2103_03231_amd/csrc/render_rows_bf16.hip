// render_rows_bf16.hip - render kernels with bf16 networks and tiles of 32 or 64
// rays, for calls that do not fill the chip with the main kernel's tiles; top-N
// and inverse-CDF placement, both depth-network inputs.
#include "rows_kernel.h"

namespace donerf {

hipError_t launch_rows_bf16(int cdf, int ncap, int din, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    return a.tile_rays == 32   ? launch_rows<kBF16, 1>(cdf, ncap, din, a, grid, stream)
           : a.tile_rays == 64 ? launch_rows<kBF16, 2>(cdf, ncap, din, a, grid, stream)
                               : hipErrorInvalidValue;   // no such tile
}

}  // namespace donerf
