// A triangle's fixed-point setup record and the raster's sample tests on it.
// The functions run on the host too, where they are tested over the whole range
// of coordinates that the setup admits.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace dsm {

constexpr int kSub = 256;              // 8 sub-pixel bits of the fixed-point grid
constexpr uint64_t kBgKey = ~0ull;     // background key (no triangle)

// Per (view, triangle) fixed-point setup, written by the setup kernel.
struct TriSetup {
    long long A;                 // doubled area, > 0 when valid
    int X[3], Y[3];              // oriented fixed-point screen coordinates
    float z[3];                  // oriented z01
    unsigned short bx0, by0, bx1, by1;  // inclusive pixel bbox, clipped to the view
    signed char facing;          // +1 / -1 orientation before re-orienting, 0 if not rasterized
    unsigned char swapped;       // 2nd and 3rd vertex exchanged
    unsigned char pad1[2];
    int pad2[2];                 // view, 0
};
static_assert(sizeof(TriSetup) == 64, "TriSetup must stay 64 bytes");

// A triangle as the raster tests it: the edge functions of edges 1 and 2 in
// plane form, E_e(px, py) = a px + b py + c with a = -dy, b = dx,
// c = dy xa - dx ya for the directed edge a -> b opposite vertex e, and
// E_0 = A - E_1 - E_2 (the three sub-triangles' doubled areas sum to A at
// every point).  With fixed-point coordinates below 2^23 and differences
// below 2^24 every term and every partial sum is an integer below 2^50, so
// float64 holds the coefficients and evaluates the functions exactly: the
// same value, and the same inside / top-left / depth results, as the 64-bit
// integer form.  The constants hold E_e - 1 for edges that are neither top
// nor left: E_e is an integer, so "E_e > 0, or E_e = 0 on a top or left edge"
// is "not negative" for the stored form, and one sign test decides all three.
// The constants are relative to an origin in whole pixels (a tile's first).
struct RasterTri {
    double c1, c2, A;       // E_1, E_2 at the origin and the doubled area, less their edges' 1 or 0
    int a1, b1, a2, b2;
    float z0, dz1, dz2;     // z0, z1 - z0, z2 - z0
    float rA;               // correctly rounded float32 1 / A
    unsigned tri;
    unsigned box;           // x0 | x1 << 5 | y0 << 10 | y1 << 15 (samples of its tile) | tile << 20 | edge bits << 24
};
static_assert(sizeof(RasterTri) == 64, "RasterTri is four 16-byte LDS words");
constexpr unsigned kTL1 = 1u << 24, kTL2 = 1u << 25;       // edge 1 / 2 is a top or left edge

__host__ __device__ __forceinline__ bool top_left(int xa, int ya, int xb, int yb) {
    const int dx = xb - xa, dy = yb - ya;
    return dy < 0 || (dy == 0 && dx > 0);
}

// The record of triangle s relative to pixel (ox, oy); box holds the edge bits only.
__host__ __device__ __forceinline__ RasterTri load_raster_tri(const TriSetup &s, unsigned local, int ox, int oy) {
    RasterTri r;
    const double px = (double)(ox * kSub), py = (double)(oy * kSub);
    const bool tl0 = top_left(s.X[1], s.Y[1], s.X[2], s.Y[2]), tl1 = top_left(s.X[2], s.Y[2], s.X[0], s.Y[0]),
               tl2 = top_left(s.X[0], s.Y[0], s.X[1], s.Y[1]);
    r.a1 = s.Y[2] - s.Y[0];
    r.b1 = s.X[0] - s.X[2];
    r.a2 = s.Y[0] - s.Y[1];
    r.b2 = s.X[1] - s.X[0];
    const double t0 = tl0 ? 0.0 : 1.0, t1 = tl1 ? 0.0 : 1.0, t2 = tl2 ? 0.0 : 1.0;
    // E_1 = a1 (px - X2) + b1 (py - Y2), E_2 = a2 (px - X0) + b2 (py - Y0)
    r.c1 = fma((double)r.a1, px - (double)s.X[2], fma((double)r.b1, py - (double)s.Y[2], -t1));
    r.c2 = fma((double)r.a2, px - (double)s.X[0], fma((double)r.b2, py - (double)s.Y[0], -t2));
    r.A = (double)s.A - ((t0 + t1) + t2);
    r.z0 = s.z[0];
    r.dz1 = s.z[1] - s.z[0];
    r.dz2 = s.z[2] - s.z[0];
    r.rA = 1.0f / (float)(double)s.A;
    r.tri = local;
    r.box = (tl1 ? kTL1 : 0u) | (tl2 ? kTL2 : 0u);
    return r;
}

__host__ __device__ __forceinline__ int high_word(double x) { return (int)(__builtin_bit_cast(uint64_t, x) >> 32); }

// Key of triangle r at a sample with edge functions (e1, e2) in the stored
// form, or kBgKey when not covered.
__host__ __device__ __forceinline__ unsigned long long edge_key(const RasterTri &r, double e1, double e2) {
    const double e0 = (r.A - e1) - e2;
    // exact sums of integers are never -0, so the sign bits are the test
    if ((high_word(e0) | high_word(e1) | high_word(e2)) < 0) return kBgKey;
    // b_e = f32(E_e) * (1 / A): one reciprocal per triangle, one product per sample
    const float b1 = (float)(e1 + ((r.box & kTL1) ? 0.0 : 1.0)) * r.rA;
    const float b2 = (float)(e2 + ((r.box & kTL2) ? 0.0 : 1.0)) * r.rA;
    const float z = (r.z0 + b1 * r.dz1) + b2 * r.dz2;
    if (!(z >= 0.0f && z <= 1.0f)) return kBgKey;
    const unsigned bits = __builtin_bit_cast(unsigned, z) & 0x7FFFFFFFu;
    return ((unsigned long long)bits << 32) | r.tri;
}

// ... at pixel (x, y) from the record's origin.
__host__ __device__ __forceinline__ unsigned long long pixel_key(const RasterTri &r, double px, double py) {
    return edge_key(r, fma((double)r.a1, px, fma((double)r.b1, py, r.c1)),
                    fma((double)r.a2, px, fma((double)r.b2, py, r.c2)));
}
__host__ __device__ __forceinline__ double sample_pos(int i) { return (double)(i * kSub + kSub / 2); }

// False when the triangle misses every sample of the box [x0, x1] x [y0, y1]:
// some edge function is negative at the box's best corner.
__host__ __device__ __forceinline__ bool touches(const RasterTri &r, int x0, int x1, int y0, int y1) {
    const double pl = sample_pos(x0), pr = sample_pos(x1), pt = sample_pos(y0), pb = sample_pos(y1);
    const int a0 = -(r.a1 + r.a2), b0 = -(r.b1 + r.b2);
    const double c0 = (r.A - r.c1) - r.c2;
    const double m0 = fma((double)a0, a0 > 0 ? pr : pl, fma((double)b0, b0 > 0 ? pb : pt, c0));
    const double m1 = fma((double)r.a1, r.a1 > 0 ? pr : pl, fma((double)r.b1, r.b1 > 0 ? pb : pt, r.c1));
    const double m2 = fma((double)r.a2, r.a2 > 0 ? pr : pl, fma((double)r.b2, r.b2 > 0 ? pb : pt, r.c2));
    return (high_word(m0) | high_word(m1) | high_word(m2)) >= 0;
}

// f(p, key) for every covered sample of the box [x0, x1] x [y0, ...] of `area`
// samples, p = row + x in the tile's rows of T, row the box's first; one sample
// after the other, the edge functions stepped along the rows.  A step is 256 a
// or 256 b, up to 2^32: past an int, so the product is formed in float64 (exact,
// as the sums are).
template <int T, class P, class F>
__host__ __device__ __forceinline__ void step_box(const RasterTri &r, int x0, int x1, int y0, int area, P row, F f) {
    const double px = sample_pos(x0), py = sample_pos(y0);
    double r1 = fma((double)r.a1, px, fma((double)r.b1, py, r.c1));
    double r2 = fma((double)r.a2, px, fma((double)r.b2, py, r.c2));
    const double ax1 = (double)r.a1 * kSub, ax2 = (double)r.a2 * kSub;
    const double by1 = (double)r.b1 * kSub, by2 = (double)r.b2 * kSub;
    double e1 = r1, e2 = r2;
    int x = x0;
    for (int q = 0; q < area; ++q) {
        const unsigned long long key = edge_key(r, e1, e2);
        if (key != kBgKey) f(row + x, key);
        e1 += ax1;
        e2 += ax2;
        if (++x > x1) {
            x = x0;
            row += T;
            r1 += by1;
            r2 += by2;
            e1 = r1;
            e2 = r2;
        }
    }
}

}  // namespace dsm
