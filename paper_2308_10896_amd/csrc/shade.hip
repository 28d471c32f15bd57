// Forward shading kernels: moment resolve of the light views, edge smoothing
// (light maps and camera images), and the deferred Chebyshev + Lambert pass.
//
// Moment resolve (Alg. 1, RenderScene): for each shadow-map texel the world
// point x on the nearest triangle is recovered from perspective-correct
// barycentrics (the point of the triangle that projects to the texel
// centre), its distance d(x) to the light (Sec. 3: Euclidean for point and
// spot lights, from a plane outside the scene for directional lights) is
// normalized, z = d / far, and (z, z^2) is written; texels without a triangle
// hold the far value (1, 1).
//
// Lookup (Alg. 2, ComputeVisibility, and Lambert shading summed over lights):
// per camera pixel the world point x and face normal n are recovered the same
// way; per light u = L(x), (m1, m2) is fetched bilinearly (clamp-to-edge),
// sigma^2 = max(m2 - m1^2, min_variance), v = 1 if z <= m1 else
// sigma^2 / (sigma^2 + (z - m1)^2) (one-sided Chebyshev, Sec. 3); points outside
// the light frustum count as lit; colour = albedo * sum_l max(0, n.omega_l)
// v_l I_l cone_l.
#include "aa.h"
#include "dsm_internal.h"

namespace dsm {

// Pixels per thread of the lookup (latency hiding; see lookup_kernel).
constexpr int kLookupPixelsPerThread = 2;

struct Bary {
    float b0, b1, b2;
};

// Barycentrics of the point of triangle (c0, c1, c2) that projects to NDC
// (px, py): sum b_i (x_i - px w_i) = 0, sum b_i (y_i - py w_i) = 0, sum b_i = 1,
// through the hardware reciprocal of the sum (about one ulp; the resolve, the
// lookup and their adjoints all form them this way).
__device__ __forceinline__ Bary persp_bary_rcp(float4 c0, float4 c1, float4 c2, float px, float py) {
    const float a0x = c0.x - px * c0.w, a0y = c0.y - py * c0.w;
    const float a1x = c1.x - px * c1.w, a1y = c1.y - py * c1.w;
    const float a2x = c2.x - px * c2.w, a2y = c2.y - py * c2.w;
    const float k0 = a1x * a2y - a1y * a2x;
    const float k1 = a2x * a0y - a2y * a0x;
    const float k2 = a0x * a1y - a0y * a1x;
    const float rs = __builtin_amdgcn_rcpf(k0 + k1 + k2);
    return Bary{k0 * rs, k1 * rs, k2 * rs};
}

// The resolve and the lookup form their quotients through the hardware
// reciprocal (about 1 ulp), where the raster setup, whose coverage and depth
// keys are integer results, keeps the correctly rounded division.  The
// lookup's adjoint forms every value with the same expressions (the map
// position, which picks the bilinear cell and the inside test, among them),
// so the two passes take the same decisions.
__device__ __forceinline__ float ndc_centre(int i, int n) {
    return (float)(2 * i + 1) * __builtin_amdgcn_rcpf((float)n) - 1.0f;
}

__device__ __forceinline__ float light_depth(const ViewConst &l, float x, float y, float z) {
    float d;
    if (l.kind == kDirectional) {
        d = ((x - l.pos[0]) * l.dir[0] + (y - l.pos[1]) * l.dir[1]) + (z - l.pos[2]) * l.dir[2];
    } else {
        const float dx = x - l.pos[0], dy = y - l.pos[1], dz = z - l.pos[2];
        d = sqrtf((dx * dx + dy * dy) + dz * dz);
    }
    return d * __builtin_amdgcn_rcpf(l.zfar) - l.zc;
}

// ----------------------------------------------------------------------------- light moments

// f of a light-map texel (i, j) with the given key: z - zc of the nearest
// triangle's point, or exp(c (z - zc)) for exponential maps.
__device__ __forceinline__ float texel_moment(const ViewConst &l, const TriVerts &r, unsigned long long key, int i,
                                              int j) {
    const int S = l.W;
    float z = 1.0f - l.zc;          // background: the far plane
    if (key != kBgKey) {
        const float v0[3] = {r.a.x, r.a.y, r.a.z}, v1[3] = {r.a.w, r.b.x, r.b.y}, v2[3] = {r.b.z, r.b.w, r.c.x};
        const float px = ndc_centre(i, S), py = -ndc_centre(j, S);
        const float4 c0 = clip_of(l.M, v0[0], v0[1], v0[2]), c1 = clip_of(l.M, v1[0], v1[1], v1[2]),
                     c2 = clip_of(l.M, v2[0], v2[1], v2[2]);
        const Bary b = persp_bary_rcp(c0, c1, c2, px, py);
        const float x = (b.b0 * v0[0] + b.b1 * v1[0]) + b.b2 * v2[0];
        const float y = (b.b0 * v0[1] + b.b1 * v1[1]) + b.b2 * v2[1];
        const float zz = (b.b0 * v0[2] + b.b1 * v1[2]) + b.b2 * v2[2];
        z = light_depth(l, x, y, zz);
    }
    return l.warp_c > 0.f ? expf(l.warp_c * z) : z;     // exponential maps
}

// Moment resolve and edge smoothing of the light maps: a wave per 64 x 4
// region, four texels a lane with their keys, then their face records, in
// flight together.  F0 keeps f alone (f^2 is its square); F1 takes the
// smoothed (f, f^2).  A pair's giving sample outside the region is resolved
// again from its key.  Bytes a texel: 8 (key) + 4 (F0) + 8 (F1) + 1 (flag),
// where a resolve, a copying pass and a list pass moved 41; 64 512^2 maps
// 212 -> 119 us (vector issue and the record gathers; the bytes take 70),
// three 2048^2 maps 177 -> 88.  At 6 waves per SIMD (5 and 8, which spills, were
// 6 and 60 % slower), the XCDs in turns of 16 regions (127 and 100 with a range
// each).
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6))) void light_moments_kernel(const ViewConst *__restrict__ views,
                                                           const TriVerts *__restrict__ tv,
                                                           const TriSetup *__restrict__ setup,
                                                           const int *__restrict__ faces,
                                                           const unsigned char *__restrict__ silm,
                                                           const float *__restrict__ verts,
                                                           const unsigned long long *__restrict__ keys,
                                                           float *__restrict__ F0, float *__restrict__ F1,
                                                           unsigned char *__restrict__ flag) {
    constexpr int ZW = kAaW + 2;
    __shared__ AARegion g;
    __shared__ float zs[(kAaH + 2) * ZW];       // f of the region and, where a pair needs it, of its border
    const Blk blk = xcd_block2<16, 8192, true>();
    const ViewConst &l = views[blk.y];
    const int S = l.W;
    if (blk.x >= aa_regions(S, S)) return;
    const int lane = (int)threadIdx.x, rxn = (S + kAaW - 1) / kAaW;
    const int i0 = (blk.x % rxn) * kAaW, j0 = (blk.x / rxn) * kAaH, i = i0 + lane;
    const unsigned long long *kv = keys + l.pix_off;
    const AAKeys k = aa_keys(kv, S, S, i0, j0, lane);
    TriVerts r[kAaH];
#pragma unroll
    for (int q = 0; q < kAaH; ++q)
        if (k.k[q + 1] != kBgKey) r[q] = tv[l.face_off + (int)(unsigned)k.k[q + 1]];
    float z[kAaH];
    float *f0 = F0 + l.map_off / 2;
#pragma unroll
    for (int q = 0; q < kAaH; ++q) {
        z[q] = texel_moment(l, r[q], k.k[q + 1], i, j0 + q);
        if (k.ok[q + 1]) f0[(j0 + q) * S + i] = z[q];
    }
    const int n = l.antialias && l.nfaces > 0 ? aa_list(g, k, silm + l.setup_off, lane) : 0;
    if (n) {
#pragma unroll
        for (int q = 0; q < kAaH; ++q) zs[(q + 1) * ZW + lane + 1] = z[q];
        __syncthreads();
        for (int e = lane; e < n; e += 64) {
            const int slot = g.item[e];
            const AASlot s = aa_slot(slot);
            const unsigned long long ka = kv[(j0 + s.ja) * S + i0 + s.ia], kb = kv[(j0 + s.jb) * S + i0 + s.ib];
            const bool front = ka < kb;
            AAPair pr{};
            if (!aa_eval<false>(l, setup, faces, silm, verts, front ? (unsigned)ka : (unsigned)kb, front, i0 + s.ia,
                                j0 + s.ja, i0 + s.ib, j0 + s.jb, s.horiz, pr))
                continue;
            const unsigned char recv = aa_receiver(pr, front);
            g.state[slot] = kAaCand | recv;
            g.w[slot] = pr.w;
            const int gi = recv == kAaA ? s.ib : s.ia, gj = recv == kAaA ? s.jb : s.ja;
            if (!aa_inside(gi, gj)) {
                const unsigned long long kg = recv == kAaA ? kb : ka;
                TriVerts t{};
                if (kg != kBgKey) t = tv[l.face_off + (int)(unsigned)kg];
                zs[(gj + 1) * ZW + gi + 1] = texel_moment(l, t, kg, i0 + gi, j0 + gj);
            }
        }
        __syncthreads();
    }
    const long long plane = (long long)S * S;
#pragma unroll
    for (int q = 0; q < kAaH; ++q) {
        if (!k.ok[q + 1]) continue;
        const int p = (j0 + q) * S + i;
        const float f = z[q], ff = f * f;
        float a0 = f, a1 = ff;
        unsigned any = 0;
        if (n)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int slot = aa_slot_of(lane, q, d);
                const unsigned st = g.state[slot];
                any |= st;
                if (!(st & aa_self_bit(d))) continue;
                const float fn = zs[(q + 1 + (d == 2 ? -1 : d == 3 ? 1 : 0)) * ZW + lane + 1 +
                                    (d == 0 ? -1 : d == 1 ? 1 : 0)];
                a0 += g.w[slot] * (fn - f);
                a1 += g.w[slot] * (fn * fn - ff);
            }
        F1[l.map_off + p] = a0;
        F1[l.map_off + plane + p] = a1;
        flag[l.pix_off + p] = any ? 1 : 0;       // for the adjoint: this sample has candidate pairs
    }
}

// ----------------------------------------------------------------------------- camera smoothing

// Edge smoothing of the camera images, a wave per 64 x 4 region, for a chunk
// of the camera's renders: the pairs depend on the keys alone, so they are
// evaluated once for all of them.  Latency of the pairs' loads bounds it; 64
// 512^2 images 121 -> 73 us against four pair tests per thread in place, 16
// cameras with 8 renders each 211 -> 95.  One channel at 8 waves per SIMD (6:
// 77 us), three at 5 (8 spills: 22 -> 29 us on a 1080p image).
template <int C>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(C == 1 ? 8 : 5))) void aa_camera_forward_kernel(
    const ViewConst *__restrict__ views, int L, const RenderConst *__restrict__ renders,
    const int *__restrict__ cam_renders_off, const int *__restrict__ cam_renders, int chunk,
    const TriSetup *__restrict__ setup, const int *__restrict__ faces, const unsigned char *__restrict__ silm,
    const float *__restrict__ verts, const unsigned long long *__restrict__ keys, const float *__restrict__ src,
    float *__restrict__ dst, unsigned char *__restrict__ flag) {
    __shared__ AARegion g;
    const Blk blk = xcd_block2<16, 8192>();
    const ViewConst &v = views[L + blk.y];
    const int W = v.W, H = v.H;
    if (blk.x >= aa_regions(W, H)) return;
    const int r0 = cam_renders_off[blk.y] + (int)blockIdx.z * chunk, r1 = min(r0 + chunk, cam_renders_off[blk.y + 1]);
    if (r0 >= r1) return;
    const int lane = (int)threadIdx.x, rxn = (W + kAaW - 1) / kAaW;
    const int i0 = (blk.x % rxn) * kAaW, j0 = (blk.x / rxn) * kAaH, i = i0 + lane;
    long long base = renders[cam_renders[r0]].img_off;
    float self[kAaH][C];
#pragma unroll
    for (int q = 0; q < kAaH; ++q)
#pragma unroll
        for (int c = 0; c < C; ++c)
            self[q][c] = i < W && j0 + q < H ? src[base + ((long long)(j0 + q) * W + i) * C + c] : 0.f;
    int n = 0;
    if (v.antialias && v.nfaces > 0) {                          // uniform
        const unsigned long long *kv = keys + v.pix_off;
        n = aa_list(g, aa_keys(kv, W, H, i0, j0, lane), silm + v.setup_off, lane);
        for (int e = lane; e < n; e += 64) {
            const int slot = g.item[e];
            const AASlot s = aa_slot(slot);
            const unsigned long long ka = kv[(j0 + s.ja) * W + i0 + s.ia], kb = kv[(j0 + s.jb) * W + i0 + s.ib];
            const bool front = ka < kb;
            AAPair pr{};
            if (!aa_eval<false>(v, setup, faces, silm, verts, front ? (unsigned)ka : (unsigned)kb, front, i0 + s.ia,
                                j0 + s.ja, i0 + s.ib, j0 + s.jb, s.horiz, pr))
                continue;
            g.state[slot] = kAaCand | aa_receiver(pr, front);
            g.w[slot] = pr.w;
        }
        __syncthreads();
    }
    for (int r = r0;;) {
#pragma unroll
        for (int q = 0; q < kAaH; ++q) {
            if (!(i < W && j0 + q < H)) continue;
            const long long p = (long long)(j0 + q) * W + i;
            float acc[C];
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = self[q][c];
            unsigned any = 0;
            if (n)
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int slot = aa_slot_of(lane, q, d);
                    const unsigned st = g.state[slot];
                    any |= st;
                    if (!(st & aa_self_bit(d))) continue;
                    const float w = g.w[slot];
                    const long long pn = p + (d == 0 ? -1 : d == 1 ? 1 : d == 2 ? -W : W);
#pragma unroll
                    for (int c = 0; c < C; ++c) acc[c] += w * (src[base + pn * C + c] - self[q][c]);
                }
#pragma unroll
            for (int c = 0; c < C; ++c) dst[base + p * C + c] = acc[c];
            if (r == r0 && blockIdx.z == 0) flag[v.pix_off + p] = any ? 1 : 0;      // for the adjoint
        }
        if (++r >= r1) break;
        base = renders[cam_renders[r]].img_off;
#pragma unroll
        for (int q = 0; q < kAaH; ++q)
#pragma unroll
            for (int c = 0; c < C; ++c)
                self[q][c] = i < W && j0 + q < H ? src[base + ((long long)(j0 + q) * W + i) * C + c] : 0.f;
    }
}

// ----------------------------------------------------------------------------- lookup + shade

// PPT pixels per thread, PPT * 256 contiguous pixels per workgroup (pixel
// k of a thread at k * 256 + its lane, so every load stays coalesced).  The
// three dependent gathers of a pixel (its depth|id key, its triangle's
// record, its map taps) are issued for all PPT pixels before any of them is
// used, so a thread waits for three round trips per PPT pixels instead of
// three per pixel.  The pixels' points and normals are formed once for a chunk
// of the camera's renders.  Each pixel's arithmetic is the one-pixel form,
// unchanged.
template <int PPT>
__global__ __launch_bounds__(256) void lookup_kernel(const ViewConst *__restrict__ views, int L,
                                                     const RenderConst *__restrict__ renders,
                                                     const int *__restrict__ cam_renders_off,
                                                     const int *__restrict__ cam_renders, int chunk,
                                                     const int *__restrict__ render_lights,
                                                     const TriVerts *__restrict__ tv,
                                                     const unsigned long long *__restrict__ keys,
                                                     const float *__restrict__ maps, float *__restrict__ img0, int C) {
    const int r0 = cam_renders_off[blockIdx.y] + (int)blockIdx.z * chunk,
              r1 = min(r0 + chunk, cam_renders_off[blockIdx.y + 1]);
    if (r0 >= r1) return;
    const ViewConst &cv = views[L + blockIdx.y];
    const int W = cv.W, H = cv.H, P = W * H;
    const int p0 = blockIdx.x * (256 * PPT) + (int)threadIdx.x;
    if (p0 >= P) return;
    unsigned long long key[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int p = p0 + 256 * k;
        key[k] = p < P ? keys[cv.pix_off + p] : kBgKey;
    }
    TriVerts r[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k)
        if (key[k] != kBgKey) r[k] = tv[cv.face_off + (int)(unsigned)key[k]];
    float x[PPT], y[PPT], z[PPT], nx[PPT], ny[PPT], nz[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        x[k] = y[k] = z[k] = nx[k] = ny[k] = nz[k] = 0.f;
        if (key[k] == kBgKey) continue;
        const float v0[3] = {r[k].a.x, r[k].a.y, r[k].a.z}, v1[3] = {r[k].a.w, r[k].b.x, r[k].b.y},
                    v2[3] = {r[k].b.z, r[k].b.w, r[k].c.x};
        const int p = p0 + 256 * k;
        const int i = p % W, j = p / W;
        const float px = ndc_centre(i, W), py = -ndc_centre(j, H);
        const float4 c0 = clip_of(cv.M, v0[0], v0[1], v0[2]), c1 = clip_of(cv.M, v1[0], v1[1], v1[2]),
                     c2 = clip_of(cv.M, v2[0], v2[1], v2[2]);
        const Bary b = persp_bary_rcp(c0, c1, c2, px, py);
        x[k] = (b.b0 * v0[0] + b.b1 * v1[0]) + b.b2 * v2[0];
        y[k] = (b.b0 * v0[1] + b.b1 * v1[1]) + b.b2 * v2[1];
        z[k] = (b.b0 * v0[2] + b.b1 * v1[2]) + b.b2 * v2[2];
        const float e1x = v1[0] - v0[0], e1y = v1[1] - v0[1], e1z = v1[2] - v0[2];
        const float e2x = v2[0] - v0[0], e2y = v2[1] - v0[1], e2z = v2[2] - v0[2];
        float cx = e1y * e2z - e1z * e2y, cy = e1z * e2x - e1x * e2z, cz = e1x * e2y - e1y * e2x;
        const float rn = __builtin_amdgcn_rsqf((cx * cx + cy * cy) + cz * cz);
        nx[k] = cx * rn;
        ny[k] = cy * rn;
        nz[k] = cz * rn;
    }
    for (int rr = r0; rr < r1; ++rr) {
        const RenderConst &R = renders[cam_renders[rr]];
        float shade[PPT];
#pragma unroll
        for (int k = 0; k < PPT; ++k) shade[k] = 0.f;
        for (int q = 0; q < R.light_count; ++q) {
            const ViewConst &l = views[render_lights[R.light_begin + q]];
            const int S = l.W, Sp = S + 2 * l.fpad;
            const float2 *mm = (const float2 *)(maps + l.fmap_off);     // (m1, m2) interleaved per texel
            bool inside[PPT];
            float fx[PPT], fy[PPT];
            int o00[PPT], o01[PPT], o10[PPT], o11[PPT];
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                inside[k] = false;
                fx[k] = fy[k] = 0.f;
                o00[k] = o01[k] = o10[k] = o11[k] = 0;
                if (key[k] == kBgKey) continue;
                // a cube face lights only the directions it owns: no fetch elsewhere
                if (l.kind == kCubeFace &&
                    cube_face_of(x[k] - l.pos[0], y[k] - l.pos[1], z[k] - l.pos[2]) != l.cube_face)
                    continue;
                const float *M = l.M;
                const float cx = ((M[0] * x[k] + M[1] * y[k]) + M[2] * z[k]) + M[3];
                const float cy = ((M[4] * x[k] + M[5] * y[k]) + M[6] * z[k]) + M[7];
                const float cw = ((M[12] * x[k] + M[13] * y[k]) + M[14] * z[k]) + M[15];
                const float rcw = __builtin_amdgcn_rcpf(cw);
                const float ux = cx * rcw, uy = cy * rcw;
                inside[k] = cw > 0.f && fabsf(ux) <= 1.f && fabsf(uy) <= 1.f;
                if (!inside[k]) continue;
                const float sx = (ux + 1.f) * (0.5f * S) - 0.5f;
                const float sy = (1.f - uy) * (0.5f * S) - 0.5f;
                const float fx0 = floorf(sx), fy0 = floorf(sy);
                fx[k] = sx - fx0;
                fy[k] = sy - fy0;
                const int ix = (int)fx0 + l.fpad, iy = (int)fy0 + l.fpad;
                const int x0 = min(max(ix, 0), Sp - 1), x1 = min(max(ix + 1, 0), Sp - 1);
                const int y0 = min(max(iy, 0), Sp - 1), y1 = min(max(iy + 1, 0), Sp - 1);
                o00[k] = y0 * Sp + x0; o01[k] = y0 * Sp + x1;
                o10[k] = y1 * Sp + x0; o11[k] = y1 * Sp + x1;
            }
            float2 t00[PPT], t01[PPT], t10[PPT], t11[PPT];
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                // offsets of pixels without a fetch are 0, a texel of this map
                t00[k] = mm[o00[k]]; t01[k] = mm[o01[k]]; t10[k] = mm[o10[k]]; t11[k] = mm[o11[k]];
            }
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                if (key[k] == kBgKey) continue;
                if (l.kind == kCubeFace &&
                    cube_face_of(x[k] - l.pos[0], y[k] - l.pos[1], z[k] - l.pos[2]) != l.cube_face)
                    continue;
                float vis = 1.f;
                if (inside[k]) {
                    const float w00 = (1.f - fx[k]) * (1.f - fy[k]), w01 = fx[k] * (1.f - fy[k]);
                    const float w10 = (1.f - fx[k]) * fy[k], w11 = fx[k] * fy[k];
                    const float m1 = ((w00 * t00[k].x + w01 * t01[k].x) + w10 * t10[k].x) + w11 * t11[k].x;
                    const float m2 = ((w00 * t00[k].y + w01 * t01[k].y) + w10 * t10[k].y) + w11 * t11[k].y;
                    float zw, floor_v;
                    warp_receiver(l, light_depth(l, x[k], y[k], z[k]), zw, floor_v);
                    const float var = fmaxf(m2 - m1 * m1, floor_v);
                    const float dd = zw - m1;
                    vis = bleed_reduce(l, (zw <= m1) ? 1.f : var * __builtin_amdgcn_rcpf(var + dd * dd));
                }
                float ox, oy, oz;
                if (l.kind == kDirectional) {
                    ox = -l.dir[0];
                    oy = -l.dir[1];
                    oz = -l.dir[2];
                } else {
                    ox = l.pos[0] - x[k];
                    oy = l.pos[1] - y[k];
                    oz = l.pos[2] - z[k];
                    const float ron = __builtin_amdgcn_rsqf((ox * ox + oy * oy) + oz * oz);
                    ox *= ron;
                    oy *= ron;
                    oz *= ron;
                }
                const float lam = fmaxf((nx[k] * ox + ny[k] * oy) + nz[k] * oz, 0.f);
                float cone = 1.f;
                if (l.kind == kSpot) {
                    // cos of the angle between x - p and the axis: (-omega) . axis
                    const float ca = -((ox * l.dir[0] + oy * l.dir[1]) + oz * l.dir[2]);
                    cone = ca >= l.cos_half ? 1.f : 0.f;
                }
                shade[k] += lam * vis * l.intensity * cone;
            }
        }
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const int p = p0 + 256 * k;
            if (p >= P) continue;
            float *out = img0 + R.img_off + (long long)p * C;
            const float rho[3] = {r[k].c.y, r[k].c.z, r[k].c.w};    // albedo, carried in the face record
            for (int c = 0; c < C; ++c) out[c] = key[k] == kBgKey ? 0.f : rho[c] * shade[k];
        }    }
}

// ----------------------------------------------------------------------------- launchers

hipError_t launch_light_moments(const ViewConst *views, int L, int max_regions, const TriVerts *tv,
                                const TriSetup *setup, const int *faces, const unsigned char *silm, const float *verts,
                                const unsigned long long *keys, float *F0, float *F1, unsigned char *aa_flag,
                                hipStream_t s) {
    if (L == 0) return hipSuccess;
    hipLaunchKernelGGL(light_moments_kernel, dim3(max_regions, L), dim3(64), 0, s, views, tv, setup, faces, silm, verts,
                       keys, F0, F1, aa_flag);
    return hipGetLastError();
}

hipError_t launch_aa_camera(const ViewConst *views, int L, int Cm, int max_regions, int max_renders,
                            const RenderConst *renders, const int *cam_renders_off, const int *cam_renders,
                            const TriSetup *setup, const int *faces, const unsigned char *silm, const float *verts,
                            const unsigned long long *keys, const float *src, float *dst, int C,
                            unsigned char *aa_flag, hipStream_t s) {
    if (Cm == 0 || max_renders == 0) return hipSuccess;
    const int chunk = render_chunk(max_renders, (long long)max_regions * Cm);
    const dim3 grid(max_regions, Cm, (max_renders + chunk - 1) / chunk);
#define DSM_AAC(CC)                                                                                                 \
    hipLaunchKernelGGL(aa_camera_forward_kernel<CC>, grid, dim3(64), 0, s, views, L, renders, cam_renders_off,     \
                       cam_renders, chunk, setup, faces, silm, verts, keys, src, dst, aa_flag)
    if (C == 1) DSM_AAC(1);
    else DSM_AAC(3);
#undef DSM_AAC
    return hipGetLastError();
}

hipError_t launch_lookup(const ViewConst *views, int L, int Cm, int max_pix, int max_renders,
                         const RenderConst *renders, const int *cam_renders_off, const int *cam_renders,
                         const int *render_lights, const TriVerts *tv, const unsigned long long *keys,
                         const float *maps, float *img0, int C, hipStream_t s) {
    if (Cm == 0 || max_renders == 0) return hipSuccess;
    constexpr int PPT = kLookupPixelsPerThread;
    const int bx = (max_pix + 256 * PPT - 1) / (256 * PPT);
    const int chunk = render_chunk(max_renders, (long long)bx * Cm);
    hipLaunchKernelGGL(lookup_kernel<PPT>, dim3(bx, Cm, (max_renders + chunk - 1) / chunk), dim3(256), 0, s, views, L,
                       renders, cam_renders_off, cam_renders, chunk, render_lights, tv, keys, maps, img0, C);
    return hipGetLastError();
}

}  // namespace dsm
