// render_rows_bf16.hip - render kernels with bf16 networks and tiles of 32 or 64
// rays, for calls that do not fill the chip with the main kernel's tiles; top-N
// and inverse-CDF placement, both depth-network inputs.
#include "rows_kernel.h"

namespace donerf {

hipError_t launch_rows_bf16(int cdf, int ncap, int din, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    if (a.tile_rays == 32)
        return cdf ? launch_rows<kBF16, 1, true>(ncap, din, a, grid, stream)
                   : launch_rows<kBF16, 1, false>(ncap, din, a, grid, stream);
    if (a.tile_rays != 64) return hipErrorInvalidValue;   // no such tile
    return cdf ? launch_rows<kBF16, 2, true>(ncap, din, a, grid, stream)
               : launch_rows<kBF16, 2, false>(ncap, din, a, grid, stream);
}

}  // namespace donerf
