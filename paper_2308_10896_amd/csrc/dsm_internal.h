// Internal layout shared by the HIP translation units of the library.
// Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dsm.h"
#include "raster_tri.h"
#include "xcd_order.h"

namespace dsm {

constexpr float kGuard = 32768.0f;     // |screen coordinate| limit in pixels
constexpr int kMaxTaps = 32;

enum ViewKind { kDirectional = 0, kPoint = 1, kSpot = 2, kCamera = 3, kCubeFace = 4 };

// One view: a light camera (views [0, L)) or a viewer camera (views [L, L+Cm)).
// Light views get M / pos / dir rewritten on the device by every forward.
struct ViewConst {
    float M[16];        // row-major view-projection, clip = M [x, 1]
    float pos[3];       // point/spot: position; directional: eye
    float dir[3];       // directional: unit travel direction; spot: cone axis
    float zfar;         // distance normalization
    float cos_half;     // spot cone
    float intensity;
    float min_var;
    int kind;
    int scene;
    int W, H;
    int vert_off, nverts;
    int face_off, nfaces;
    int clip_off;       // first vertex of this view in the clip / gclip arrays
    int setup_off;      // first triangle of this view in the per-(view, triangle) arrays
    long long pix_off;  // first sample of this view in the key array
    int tile_off;       // first tile of this view in the global tile list
    int tiles_x, tiles_y;
    int antialias;
    long long map_off;  // light views: first texel of the 2-channel maps (plane stride S*S)
    int part_off;       // light views: first per-tile slot of the backward light-frame partials
    int part_gm_off;    // light views: first slot of the dL/dM partials (one per 64 vertices)
    int cube_face;      // cube-face lights: face 0..5 (+x, -x, +y, -y, +z, -z)
    float warp_c;       // light views: exponential maps store exp(c z), exp(2 c z); 0 = plain z, z^2
    float bleed;        // light views: light-bleeding reduction amount
    long long fmap_off; // light views: first texel of the filtered maps (and their gradient), side W + 2 fpad
    long long pad_off;  // cube faces: first texel of the padded unfiltered maps in the smoothed-map buffers
    int fpad;           // cube faces: texels of padding sampled from the neighbouring faces; else 0
    int cube_nb[4];     // cube faces, per map edge (left, right, top, bottom): neighbour face
                        // | its edge << 3 | (indices along the edge reversed) << 5
    int ring_off;       // cube faces: first CubeTap of this face's padding (4 P S entries)
    float zc;           // light views: reference depth; maps hold moments of z - zc (see light_depth)
    int write_tv;       // first view of its scene: its setup writes the scene's TriVerts records
    int tri_block;      // first TriBlock of this view
};

// A run of triangles of one view, a workgroup's share of the triangle passes.
struct TriBlock {
    int view, first;
};
// The totals of a triangle pass's workgroups are also added up by groups, and
// up to kMaxTriGroups groups every workgroup sums those before it; the large
// triangles' workgroups hold the groups' prefix in LDS.
constexpr int kTriRun = 256, kTriGroup = 64, kMaxTriGroups = 1024;
// Group totals lie a cache line apart: their atomics meet only within a group
// (side by side the setup of 99k triangles in 24 views took 79 us, not 66).
constexpr int kGroupStride = 16;      // of 8 bytes
// Pairs are numbered in 32 bits, and the bins hold fewer than 2^28, but many
// triangles over whole large views (an optimization that diverged) have more
// than 2^32 of them: the number stays at kPairEnd from there on, so that every
// triangle past the bins stays past them.
constexpr unsigned kPairEnd = 0x7fffffffu;
__device__ __forceinline__ unsigned add_sat(unsigned a, unsigned b) { return __builtin_elementwise_add_sat(a, b); }
__device__ __forceinline__ unsigned word_sat(unsigned long long x) { return x >> 32 ? ~0u : (unsigned)x; }
// Tiles per workgroup of the tile scan.
constexpr int kScanShift = 11, kScanBlock = 1 << kScanShift;

// One padded texel of a cube face beyond one of its edges: the bilinear
// sample of the neighbouring face g along the direction the padded texel
// centre looks along.  Entries of a face run over edge e (left, right, top,
// bottom), depth k = 1..P beyond it, and position t = 0..S-1 along it.
struct CubeTap {
    int g;                        // neighbouring face 0..5
    int o[4];                     // texel indices j * S + i of the taps in g's map
    float w[4];                   // bilinear weights (clamp-to-edge taps)
};

// Receiver depth as the lookup compares it, and the variance floor:
// exponential maps compare exp(c z) and floor sigma^2 at min_var (c exp(c z))^2
// (the floor follows the warp's slope); plain maps use z and min_var.
__device__ __forceinline__ void warp_receiver(const ViewConst &l, float zz, float &zw, float &floor_v) {
    if (l.warp_c > 0.f) {
        zw = expf(l.warp_c * zz);
        const float s = l.warp_c * zw;
        floor_v = l.min_var * (s * s);
    } else {
        zw = zz;
        floor_v = l.min_var;
    }
}

// Light-bleeding reduction: v -> clamp((v - a) / (1 - a), 0, 1) for a > 0.
__device__ __forceinline__ float bleed_reduce(const ViewConst &l, float v) {
    return l.bleed > 0.f ? fminf(fmaxf((v - l.bleed) / (1.f - l.bleed), 0.f), 1.f) : v;
}

// Cube face owning the direction d from an omnidirectional light: the axis of
// the largest |d_a| (the first one on ties) and its sign, face 2a (+) or
// 2a + 1 (-).
__device__ __forceinline__ int cube_face_of(float dx, float dy, float dz) {
    const float ax = fabsf(dx), ay = fabsf(dy), az = fabsf(dz);
    int a = 0;
    float m = ax, s = dx;
    if (ay > m) { a = 1; m = ay; s = dy; }
    if (az > m) { a = 2; s = dz; }
    return 2 * a + (s < 0.f ? 1 : 0);
}

struct RenderConst {
    int camera_view;    // view index of the camera
    int light_begin;    // range into the device list of light view indices
    int light_count;
    int W, H;
    int part_off;       // first float of this render's per-(light, tile) backward partials
    long long img_off;  // first float of the [H,W,C] image
    long long pix_off;  // camera view's first sample (keys)
};

// The light gradient's inputs and outputs: the partials of light tiles and of
// render tiles, where light_partials leaves its kGlightBlocks sums per light,
// the scenes' counters of finished workgroups, and the gradient [L][3].
struct LightSum {
    const RenderConst *renders;
    const int *light_renders_off, *light_renders;
    const float *part_light, *part_render;
    float *gl_part;
    unsigned *done;
    float *gparams;
};

// Workgroups per light in the first pass of the light-gradient reduction.
constexpr int kGlightBlocks = 16;

struct BlurJob {
    int S;
    int k;
    long long in_off;            // first float of the 2-channel input map
    long long out_off;
    int tile_off;                // first tile of this job
    int tiles_x;
    float w[kMaxTaps];
};

// Counters written by the device, read by dsm_get_stats.
struct DevCounters {
    unsigned long long culled;
    unsigned long long pairs;
    unsigned long long overflow;
    unsigned long long bad_indices;
    unsigned long long item_len;     // items of the large triangles (LargeLists)
    unsigned int overflow_list_len;
    unsigned int large_len;          // listed large triangles
    unsigned int bin_cursor;         // running total of the tile scan
    unsigned int medium_len;         // listed triangles of kOwnRows + 1 .. kBigBin pairs
    unsigned int pad[2];
};
static_assert(sizeof(DevCounters) == 64, "DevCounters is a cache line");

// Triangles of more than kBigBin tiles, and their pairs in items (triangle,
// first pair within it) of kLargeChunk.  item_cap holds every item whose pairs
// can fit the bins; with more pairs than that the items may be incomplete.
constexpr unsigned kBigBin = 32, kLargeChunk = 512;
constexpr int kLargeBlocks = 512;      // workgroups that take the items
// medium lists the triangles of more than kOwnRows pairs that are not large:
// the backward sums their rows before its gathers.
constexpr unsigned kOwnRows = 4;
struct LargeLists {
    unsigned *list;
    uint2 *items;
    unsigned item_cap;
    unsigned *medium;
};

// f(t, q0, n) for workgroup b's share of the items, n the triangle's pairs
// (count(t)).  With incomplete items every workgroup walks the triangles and
// takes its chunks of each.
template <class Count, class F>
__device__ __forceinline__ void for_large_items(const LargeLists &l, const DevCounters *counters, int b, int nb,
                                                Count count, F f) {
    const unsigned long long nitems = counters->item_len;
    const unsigned nlist = counters->large_len;
    if (nitems <= l.item_cap) {
        for (unsigned o = (unsigned)b; o < (unsigned)nitems; o += (unsigned)nb) f(l.items[o].x, l.items[o].y, count(l.items[o].x));
        return;
    }
    for (unsigned o = 0; o < nlist; ++o) {
        const unsigned t = l.list[o], n = count(t);
        for (unsigned k = ((unsigned)b + o) % (unsigned)nb; k * kLargeChunk < n; k += (unsigned)nb) f(t, k * kLargeChunk, n);
    }
}

// ----------------------------------------------------------------------------- helpers

// Sum over the 64 lanes of a wave, returned to every lane.  DPP moves inside
// each 16-lane row (quad swaps, then rotations by 4 and 8), then the four row
// sums are read out with v_readlane.  All 64 lanes must be active.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_mov<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_mov<0x124>(v);   // row_ror:4
    v += dpp_mov<0x128>(v);   // row_ror:8
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}

// lo summed over lane ^ 32 in the lower half of the wave, hi in the upper half
// (one swap of the halves instead of two selects and a permute through LDS);
// likewise over lane ^ 16 in even and odd rows of 16.
__device__ __forceinline__ float swap32_add(float lo, float hi) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_add(float lo, float hi) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Wave-wide sums of N <= 32 values at once by recursive halving: at each
// butterfly step every lane keeps half of its remaining values and receives
// its partner's copy of that half, until one value is left; the lanes that
// share it sum it.  Lane l returns the total of value l >> kSumShift<N>
// (0 for values >= N).  About 3 instructions per value; 10 in all for N <= 4.
// All 64 lanes must be active.
template <int N>
constexpr int kSumShift = N <= 4 ? 4 : N <= 8 ? 3 : N <= 16 ? 2 : 1;

template <int N>
__device__ __forceinline__ float wave_sum_multi(const float (&v)[N]) {
    static_assert(N >= 1 && N <= 32, "wave_sum_multi handles up to 32 values");
    constexpr int W = 64 >> kSumShift<N>;
    const int lane = (int)(threadIdx.x & 63);
    const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2;
    float a[W / 2];
#pragma unroll
    for (int j = 0; j < W / 2; ++j) a[j] = swap32_add(j < N ? v[j] : 0.f, j + W / 2 < N ? v[j + W / 2] : 0.f);
    float b[W / 4];
#pragma unroll
    for (int j = 0; j < W / 4; ++j) b[j] = swap16_add(a[j], a[j + W / 4]);
    if constexpr (W == 4) {
        float e = b[0];
        e += dpp_mov<0x128>(e);       // row_ror:8
        e += dpp_mov<0x124>(e);       // row_ror:4
        e += dpp_mov<0x4E>(e);        // quad_perm [2,3,0,1]
        return e + dpp_mov<0xB1>(e);  // quad_perm [1,0,3,2]
    } else {
        float c[W / 8];
#pragma unroll
        for (int j = 0; j < W / 8; ++j)           // partner lane ^ 8: row_ror:8 within 16-lane rows
            c[j] = (b3 ? b[j + W / 8] : b[j]) + dpp_mov<0x128>(b3 ? b[j] : b[j + W / 8]);
        if constexpr (W == 8) {
            float e = c[0];
            e += dpp_mov<0x141>(e);   // row_half_mirror: lane 7 - l of each 8
            e += dpp_mov<0x4E>(e);
            return e + dpp_mov<0xB1>(e);
        } else {
            float d[W / 16];
#pragma unroll
            for (int j = 0; j < W / 16; ++j) {    // partner lane ^ 4: from lane + 4 (row_ror:12) or lane - 4 (row_ror:4)
                const float send = b2 ? c[j] : c[j + W / 16];
                const float up = dpp_mov<0x12C>(send), down = dpp_mov<0x124>(send);
                d[j] = (b2 ? c[j + W / 16] : c[j]) + (b2 ? down : up);
            }
            float e;
            if constexpr (W == 16) e = d[0] + dpp_mov<0x4E>(d[0]);
            else e = (b1 ? d[1] : d[0]) + dpp_mov<0x4E>(b1 ? d[0] : d[1]);   // partner lane ^ 2
            return e + dpp_mov<0xB1>(e);                                     // partner lane ^ 1: plain sum
        }
    }
}

template <int CTRL>
__device__ __forceinline__ int dpp_movi(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, false);
}
// Minimum (maximum) over the 64 lanes of a wave of two unsigned 16-bit values
// packed in a word, returned to every lane.  All lanes active.
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
template <bool MAX>
__device__ __forceinline__ unsigned pk_best(unsigned a, unsigned b) {
    const ushort2v x = __builtin_bit_cast(ushort2v, a), y = __builtin_bit_cast(ushort2v, b);
    return __builtin_bit_cast(unsigned, MAX ? __builtin_elementwise_max(x, y) : __builtin_elementwise_min(x, y));
}
template <bool MAX>
__device__ __forceinline__ unsigned wave_pk_best(unsigned v) {
    v = pk_best<MAX>(v, (unsigned)dpp_movi<0xB1>((int)v));
    v = pk_best<MAX>(v, (unsigned)dpp_movi<0x4E>((int)v));
    v = pk_best<MAX>(v, (unsigned)dpp_movi<0x124>((int)v));
    v = pk_best<MAX>(v, (unsigned)dpp_movi<0x128>((int)v));
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = pk_best<MAX>(r[0], r[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (unsigned)__builtin_amdgcn_readfirstlane((int)pk_best<MAX>(q[0], q[1]));
}

// Order the LDS accesses of a wave's lanes before and after (the hardware
// keeps them in order; this keeps the compiler from carrying a value across).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (x, y) of this workgroup's item in a grid of views y (xcd_item).
struct Blk {
    int x, y;
};
template <int RUN, int FROM, bool SPREAD = false>
__device__ __forceinline__ Blk xcd_block2() {
    const int gx = (int)gridDim.x;
    const int lin = xcd_item<RUN, FROM, SPREAD>((int)blockIdx.x + (int)blockIdx.y * gx, gx, (int)gridDim.y);
    return Blk{lin % gx, lin / gx};
}

// Clip coordinates M [x, 1] in the fixed operation order every kernel uses
// (no contraction), so that recomputing them anywhere is bit-identical.
__device__ __forceinline__ float4 clip_of(const float *M, float x, float y, float z) {
    float4 c;
    c.x = ((M[0] * x + M[1] * y) + M[2] * z) + M[3];
    c.y = ((M[4] * x + M[5] * y) + M[6] * z) + M[7];
    c.z = ((M[8] * x + M[9] * y) + M[10] * z) + M[11];
    c.w = ((M[12] * x + M[13] * y) + M[14] * z) + M[15];
    return c;
}

// World positions of a triangle's three corners, packed as three float4
// (x0 y0 z0 x1 | y1 z1 x2 y2 | z2 - - -), one record per face of the batch.
struct TriVerts {
    float4 a, b, c;     // x0 y0 z0 x1 | y1 z1 x2 y2 | z2 albedo[0..2]
};

__device__ __forceinline__ void atomic_add_f32(float *p, float v) {
    if (v != 0.0f) atomicAdd(p, v);
}

}  // namespace dsm

// Host-side launchers implemented per translation unit.
namespace dsm {
hipError_t launch_blur(const BlurJob *jobs_dev, int njobs, int total_tiles, const float *in, float *out,
                       bool adjoint, int R, int ty, hipStream_t s);
// Tile height for radius R where blur_tall_tiles would sum to tall_tiles.
int blur_tile_height(int R, long long tall_tiles);
int blur_tall_tiles(int S, int R);
hipError_t launch_blur_uniform(const BlurJob &job, int n_maps, const float *in, float *out, bool adjoint,
                               hipStream_t s);
int blur_tiles(int S, int ty);
int blur_tiles_x(int S);
bool valid_filter(int S, int filter, int k);

struct CamStatic;
// Jacobian of a light frame (M[16], pos[3], dir[3]) w.r.t. its three parameter components, [22][3].
constexpr int kJac = 66;
// Also clears bytes1 at z1 and bytes2 at z2 (multiples of 4) and, with rows, the
// 96-byte rows of the listed triangles, in the same launch; with *pairs at
// kPairEnd, where a triangle's pair numbers do not say whether it has any, the
// rows of all ntri triangles.
struct ClearRows {
    float *rows;                    // nullptr: none
    const unsigned *list_a, *list_b;
    const unsigned *len_a, *len_b;
    const unsigned *pairs;
    unsigned ntri;
};
hipError_t launch_light_frames(ViewConst *views, const CamStatic *cams, const float *params, int L, float *jac,
                               float *zc_out, void *z1, size_t bytes1, void *z2, size_t bytes2, const ClearRows &rows,
                               hipStream_t s);
hipError_t launch_setup(const ViewConst *views, const TriBlock *blocks, int nblocks, const int *faces,
                        const float *verts, const float *albedo, int C, TriVerts *tv, TriSetup *setup,
                        signed char *facing8, unsigned *pair_local, unsigned *block_total,
                        unsigned long long *group_total, const LargeLists &large, int tile, DevCounters *counters, hipStream_t s);
hipError_t launch_binning(const ViewConst *views, const TriBlock *blocks, int nblocks, const TriSetup *setup,
                          const int *adj, const signed char *facing8, unsigned char *silm, const unsigned *pair_local,
                          unsigned *block_total, const unsigned long long *group_total, unsigned *pair_off,
                          int ntri, unsigned capacity, int tile,
                          unsigned *tile_count, unsigned *tile_start, unsigned *pair_slot, int ntiles, unsigned *bins,
                          unsigned *bin_pair, unsigned *overflow_list, const LargeLists &large,
                          DevCounters *counters, unsigned long long *keys, long long nkeys,
                          hipStream_t s);
hipError_t launch_raster(const ViewConst *views, const int *tile_view, int ntiles, int tile, const TriSetup *setup,
                         const unsigned *tile_start, const unsigned *bins, const unsigned *overflow_list,
                         DevCounters *counters, unsigned long long *keys, hipStream_t s);
hipError_t launch_cube_pad(const ViewConst *views, int L, int max_padded, const CubeTap *taps, float *F1,
                           hipStream_t s);
hipError_t launch_cube_pad_transpose(const ViewConst *views, int L, int max_texels, int max_ring,
                                     const CubeTap *taps, float *gF1, hipStream_t s);
hipError_t launch_light_moments(const ViewConst *views, int L, int max_regions, const TriVerts *tv,
                                const TriSetup *setup, const int *faces, const unsigned char *silm, const float *verts,
                                const unsigned long long *keys, float *F0, float *F1, unsigned char *aa_flag,
                                hipStream_t s);
hipError_t launch_aa_camera(const ViewConst *views, int L, int Cm, int max_regions, int max_renders,
                            const RenderConst *renders, const int *cam_renders_off, const int *cam_renders,
                            const TriSetup *setup, const int *faces, const unsigned char *silm, const float *verts,
                            const unsigned long long *keys, const float *src, float *dst, int C,
                            unsigned char *aa_flag, hipStream_t s);
hipError_t launch_lookup(const ViewConst *views, int L, int Cm, int max_pix, int max_renders,
                         const RenderConst *renders, const int *cam_renders_off, const int *cam_renders,
                         const int *render_lights, const TriVerts *tv, const unsigned long long *keys,
                         const float *maps, float *img0, int C, hipStream_t s);
// backward
hipError_t launch_aa_camera_backward(const ViewConst *views, int L, int Cm, int max_regions, int max_renders,
                                     const RenderConst *renders, const int *cam_renders_off, const int *cam_renders,
                                     const TriSetup *setup, const int *faces, const unsigned char *silm, const float *verts,
                                     const unsigned long long *keys, const unsigned char *aa_flag, const float *img0,
                                     const float *gimg, float *gimg0, float4 *gclip, int C, hipStream_t s);
hipError_t launch_lookup_backward(int tile, const ViewConst *views, int L, int Cm, int max_tiles,
                                  const RenderConst *renders, const int *cam_renders_off, const int *cam_renders,
                                  const int *render_lights, const TriVerts *tv, const unsigned long long *keys,
                                  const float *maps, const float *gimg0, float *gmaps, const TriSetup *setup,
                                  const unsigned *tile_start, const unsigned *bins, const unsigned *bin_pair,
                                  unsigned char *pair_flag, float *pair_sums, float *gtri, float *part_render, int C,
                                  const float *jac, const unsigned *pair_off, unsigned capacity, hipStream_t s);
hipError_t launch_light_backward(int tile, const ViewConst *views, int L, int max_tiles, const TriSetup *setup,
                                 const int *faces, const unsigned char *silm, const float *verts, const TriVerts *tv,
                                 const unsigned long long *keys, const unsigned char *aa_flag, const float *F0, const float *gF1, float4 *gclip,
                                 const unsigned *tile_start, const unsigned *bins, const unsigned *bin_pair,
                                 unsigned char *pair_flag, float *pair_sums, float *gtri, float *part_light,
                                 const float *jac, const unsigned *pair_off, unsigned capacity, hipStream_t s);
hipError_t launch_vertex_gradients(const ViewConst *views, int L, int B, int max_verts, int max_faces, int max_views,
                                   int ntri, unsigned capacity, const TriSetup *setup, const LargeLists &large,
                                   const DevCounters *counters, const int *scene_vert_off, const int *scene_face_off,
                                   const int *scene_views_off, const int *scene_views, const int *vc_off,
                                   const int *vc_list, const unsigned *pair_off, const unsigned char *pair_flag,
                                   const float *pair_sums, float *gtri, const float *zero_rec, const float *verts,
                                   const float4 *gclip, float *gverts, float *part_gm, float *galbedo, int C,
                                   const float *jac, const LightSum &ls, hipStream_t s);
hipError_t launch_pose(const int *scene_vert_off, const int *pose_counts, const float *pose_centers, int B,
                       int max_verts, const float *local, const float *poses, float *world, hipStream_t s);
hipError_t launch_pose_backward(const int *scene_vert_off, const int *pose_counts, int B, int max_verts,
                                const float *local, const float *poses, const float *gworld, float *gposes,
                                hipStream_t s);
void filter_taps_host(int filter, int k, float sigma, float *w);
}  // namespace dsm
