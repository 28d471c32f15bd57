// The stand-alone moment filter's transpose kernels (planar input).
#include "blur.h"

namespace dsm {

hipError_t launch_blur_transpose_planar(int R, int ty, dim3 grid, const BlurJob *jobs, int njobs,
                                        const BlurJob &single, int per_map, const float *in, float *out,
                                        hipStream_t s) {
    return launch_blur_radius<true, false>(R, ty, grid, jobs, njobs, single, per_map, in, out, s);
}

}  // namespace dsm
