// The raster's sample tests (csrc/raster_tri.h) compiled for the host.
#include "raster_tri.h"

// Per case: the record of a triangle relative to pixel (ox, oy) and the keys of
// its samples in the box [x0, x1] x [y0, y1] of an 8 x 8 tile there, stepped as
// a lane does alone and evaluated one by one as a wave does; touch: whether the
// box can hold a covered sample.
extern "C" void raster_tri_keys(int n, const dsm::TriSetup *tri, const int *origin, const int *box,
                                unsigned long long *stepped, unsigned long long *direct, unsigned char *touch) {
    for (int c = 0; c < n; ++c) {
        const int *b = box + 4 * c;
        const dsm::RasterTri r = dsm::load_raster_tri(tri[c], 7u, origin[2 * c], origin[2 * c + 1]);
        unsigned long long *s = stepped + 64 * c, *d = direct + 64 * c;
        for (int q = 0; q < 64; ++q) s[q] = d[q] = dsm::kBgKey;
        dsm::step_box<8>(r, b[0], b[1], b[2], (b[1] - b[0] + 1) * (b[3] - b[2] + 1), s + 8 * b[2],
                         [](unsigned long long *p, unsigned long long key) { *p = key; });
        for (int y = b[2]; y <= b[3]; ++y)
            for (int x = b[0]; x <= b[1]; ++x) d[8 * y + x] = dsm::pixel_key(r, dsm::sample_pos(x), dsm::sample_pos(y));
        touch[c] = dsm::touches(r, b[0], b[1], b[2], b[3]);
    }
}
