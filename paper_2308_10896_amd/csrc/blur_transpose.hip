// The moment filter's transpose kernels of the pipeline (interleaved input).
#include "blur.h"

namespace dsm {

hipError_t launch_blur_transpose(int R, int ty, dim3 grid, const BlurJob *jobs, int njobs, const BlurJob &single,
                                 int per_map, const float *in, float *out, hipStream_t s) {
    return launch_blur_radius<true, true>(R, ty, grid, jobs, njobs, single, per_map, in, out, s);
}

}  // namespace dsm
