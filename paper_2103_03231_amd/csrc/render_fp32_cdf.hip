// render_fp32_cdf.hip - render kernels with fp32 networks and inverse-CDF placement (Sec. 5.1),
// both depth-network inputs.  One translation unit per precision and
// placement so that the variants compile in parallel.
#include "rows_kernel.h"

namespace donerf {

hipError_t launch_render_fp32_cdf(int ncap, int din, const RenderArgs& a, dim3 grid, hipStream_t stream) {
    return launch_rows_main<kF32, kF32CB, kPlaceCdf>(ncap, din, a, grid, stream);
}

}  // namespace donerf
