// The moment filter's launchers and its forward kernels.
#include "blur.h"

#include <math.h>

namespace dsm {

int blur_tile_height(int R, long long tall_tiles) { return tall_tiles < kBlurFewTiles ? blur_short(R) : blur_tall(R); }

int blur_tiles_x(int S) { return (S + kBlurTX - 1) / kBlurTX; }
int blur_tiles(int S, int ty) { return blur_tiles_x(S) * ((S + ty - 1) / ty); }
int blur_tall_tiles(int S, int R) { return blur_tiles(S, blur_tall(R)); }

// jobs_dev: njobs jobs of one radius R (job.k == 2R + 1) and tile height ty, tile offsets from 0.
hipError_t launch_blur(const BlurJob *jobs_dev, int njobs, int total_tiles, const float *in, float *out,
                       bool adjoint, int R, int ty, hipStream_t s) {
    if (total_tiles == 0 || njobs == 0) return hipSuccess;
    BlurJob none{};
    if (adjoint) return launch_blur_transpose(R, ty, dim3(total_tiles), jobs_dev, njobs, none, 1, in, out, s);
    return launch_blur_radius<false, true>(R, ty, dim3(total_tiles), jobs_dev, njobs, none, 1, in, out, s);
}

hipError_t launch_blur_uniform(const BlurJob &job, int n_maps, const float *in, float *out, bool adjoint,
                               hipStream_t s) {
    const int R = (job.k - 1) / 2;
    BlurJob j = job;
    j.tile_off = 0;
    j.tiles_x = blur_tiles_x(job.S);
    const int ty = blur_tile_height(R, (long long)blur_tall_tiles(job.S, R) * n_maps);
    const int per_map = blur_tiles(job.S, ty);
    const long long total = (long long)per_map * n_maps;
    if (total >= (1LL << 31)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total);
    if (adjoint) return launch_blur_transpose_planar(R, ty, grid, nullptr, 0, j, per_map, in, out, s);
    return launch_blur_radius<false, false>(R, ty, grid, nullptr, 0, j, per_map, in, out, s);
}

void filter_taps_host(int filter, int k, float sigma, float *w) {
    const int r = (k - 1) / 2;
    if (filter == DSM_FILTER_BOX) {
        for (int i = 0; i < k; ++i) w[i] = (float)(1.0 / k);
        return;
    }
    double s = sigma > 0 ? (double)sigma : (k - 1) / 3.0;
    if (s <= 0) {
        w[0] = 1.f;
        return;
    }
    double acc = 0, tmp[kMaxTaps];
    for (int i = -r; i <= r; ++i) {
        tmp[i + r] = exp(-(double)(i * i) / (2.0 * s * s));
        acc += tmp[i + r];
    }
    for (int i = 0; i < k; ++i) w[i] = (float)(tmp[i] / acc);
}

}  // namespace dsm
