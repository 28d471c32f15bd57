// Reverse-mode kernels (Sec. 4: the gradient of the loss w.r.t. the scene
// parameters flows through the visibility v, the filtered moments
// m1 = G f~, m2 = G f^2~ and the smoothed shadow map; the Jacobians are never
// formed, Sec. 5).  Every kernel is the hand-written adjoint of its forward
// counterpart in shade.hip / raster.hip:
//
//   camera smoothing^T    : dL/dimage -> dL/dimage0, dL/d(clip of edge ends)
//   lookup^T              : dL/dimage0 -> dL/d(m1, m2) scattered bilinearly,
//                           dL/dvertices, dL/d(camera clip), dL/d(light frame),
//                           dL/dalbedo.  For d > mu:
//                           dv/dmu = 2 s^2 (d-mu) / (s^2+(d-mu)^2)^2 = -dv/dd
//                           (the paper's derivative, s^2 held fixed), and
//                           dv/ds^2 = (d-mu)^2 / (s^2+(d-mu)^2)^2 with
//                           s^2 = m2 - m1^2 (zero where the floor is active).
//   filter^T              : blur.hip (adjoint mode)
//   light smoothing^T + resolve^T (fused per texel)
//   transform^T           : dL/dclip -> dL/dvertices (M^T) and dL/dM
//
// Vertex-indexed gradients are reduced per (tile, triangle) before they reach
// global memory (see "tile accumulation" below).
#include <algorithm>

#include "aa.h"
#include "dsm_internal.h"
#include "frames.h"

namespace dsm {

// Scatter N values per lane to addresses that depend only on (key, i): lanes
// with equal keys are summed across the wave first.  All 64 lanes must call.
template <int N, class Addr>
__device__ __forceinline__ void scatter_by_key(bool active, int key, const float (&val)[N], Addr addr) {
    const int lane = threadIdx.x & 63;
    unsigned long long pending = __ballot(active);
    while (pending) {
        const int leader = __ffsll(pending) - 1;
        const int k = __builtin_amdgcn_readlane(key, leader);
        const bool mine = active && key == k;
        const unsigned long long m = __ballot(mine);
        pending &= ~m;
        if (__popcll(m) >= 4) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float s = wave_sum(mine ? val[i] : 0.f);
                if (lane == leader) atomic_add_f32(addr(k, i), s);
            }
        } else if (mine) {
#pragma unroll
            for (int i = 0; i < N; ++i) atomic_add_f32(addr(k, i), val[i]);
        }
    }
}

// Reciprocal (about one ulp) for gradient terms and for the shading values
// the adjoints recompute exactly as the forward kernels form them (the map
// position, which picks the bilinear cell, among them: both passes take that
// decision from the same float32 value).  The correctly rounded division,
// which the raster setup keeps for its integer results, costs about ten
// instructions, this one.
__device__ __forceinline__ float grcp(float x) { return __builtin_amdgcn_rcpf(x); }

// NDC of pixel centre i of n, as the forward resolve and lookup form it.
__device__ __forceinline__ float ndc_c(int i, int n) { return (float)(2 * i + 1) * grcp((float)n) - 1.0f; }

// Barycentrics through the hardware reciprocal of their sum (about one ulp):
// the forward lookup forms the world point the same way, so the reverse pass
// recomputes its values, and its decisions, bit for bit.
struct BaryFull {
    float a0x, a0y, a1x, a1y, a2x, a2y, k0, k1, k2, s, b0, b1, b2;
};

__device__ __forceinline__ BaryFull bary_full(float4 c0, float4 c1, float4 c2, float px, float py) {
    BaryFull r;
    r.a0x = c0.x - px * c0.w; r.a0y = c0.y - py * c0.w;
    r.a1x = c1.x - px * c1.w; r.a1y = c1.y - py * c1.w;
    r.a2x = c2.x - px * c2.w; r.a2y = c2.y - py * c2.w;
    r.k0 = r.a1x * r.a2y - r.a1y * r.a2x;
    r.k1 = r.a2x * r.a0y - r.a2y * r.a0x;
    r.k2 = r.a0x * r.a1y - r.a0y * r.a1x;
    r.s = r.k0 + r.k1 + r.k2;
    const float rs = __builtin_amdgcn_rcpf(r.s);
    r.b0 = r.k0 * rs; r.b1 = r.k1 * rs; r.b2 = r.k2 * rs;
    return r;
}

// gb (d loss / d barycentrics) -> gradient w.r.t. clip (x, y, w) of the 3 corners: out[3*i + {0,1,2}]
__device__ __forceinline__ void bary_backward(const BaryFull &b, float px, float py, float gb0, float gb1, float gb2,
                                              float out[9]) {
    // adjoint only: fused multiply-adds
    const float dotg = fmaf(gb2, b.b2, fmaf(gb1, b.b1, gb0 * b.b0));
    const float rs = grcp(b.s);
    const float gk0 = (gb0 - dotg) * rs, gk1 = (gb1 - dotg) * rs, gk2 = (gb2 - dotg) * rs;
    const float ga0x = fmaf(gk2, b.a1y, -gk1 * b.a2y), ga0y = fmaf(gk1, b.a2x, -gk2 * b.a1x);
    const float ga1x = fmaf(gk0, b.a2y, -gk2 * b.a0y), ga1y = fmaf(gk2, b.a0x, -gk0 * b.a2x);
    const float ga2x = fmaf(gk1, b.a0y, -gk0 * b.a1y), ga2y = fmaf(gk0, b.a1x, -gk1 * b.a0x);
    out[0] = ga0x; out[1] = ga0y; out[2] = -fmaf(px, ga0x, py * ga0y);
    out[3] = ga1x; out[4] = ga1y; out[5] = -fmaf(px, ga1x, py * ga1y);
    out[6] = ga2x; out[7] = ga2y; out[8] = -fmaf(px, ga2x, py * ga2y);
}

// ----------------------------------------------------------------------------- silhouette edge terms

// A silhouette pair's gradient: six terms for the clip coordinates (x, y, w)
// of its edge's two vertices.
struct EdgeTerm {
    bool has;
    int va, vb;
    float g[6];
};

__device__ __forceinline__ void edge_set(EdgeTerm &t, const AAPair &pr, double galpha) {
    galpha *= pr.recv == 1 ? 1.0 : -1.0;      // w = alpha - 1/2 or 1/2 - alpha
    t.has = true;
    t.va = pr.va;
    t.vb = pr.vb;
    t.g[0] = (float)(galpha * pr.dax);
    t.g[1] = (float)(galpha * pr.day);
    t.g[2] = (float)(galpha * pr.daw);
    t.g[3] = (float)(galpha * pr.dbx);
    t.g[4] = (float)(galpha * pr.dby);
    t.g[5] = (float)(galpha * pr.dbw);
}

// Add the lanes' terms.  Lanes with the same edge are summed in the
// wave first and added with one atomic a term: float atomics run at the
// memory side, where the hundreds of samples along a large object's outline
// would queue on the same two vertices.  All 64 lanes must call.
__device__ __forceinline__ void edge_add(EdgeTerm &t, float4 *__restrict__ gclip) {
    const int lane = (int)(threadIdx.x & 63);
    unsigned long long pending = __ballot(t.has);
    while (pending) {
        const int leader = __ffsll(pending) - 1;
        const int va = __builtin_amdgcn_readlane(t.va, leader), vb = __builtin_amdgcn_readlane(t.vb, leader);
        const bool mine = t.has && t.va == va && t.vb == vb;
        const unsigned long long m = __ballot(mine);
        pending &= ~m;
        if (__popcll(m) < 3) continue;                   // these lanes add their own below
        float v[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) v[k] = mine ? t.g[k] : 0.f;
        const float s = wave_sum_multi(v);               // lane 8k: the group's total of term k
        const int k = lane >> kSumShift<6>;
        if ((lane & 7) == 0 && k < 6) {
            float *p = (float *)(gclip + (k < 3 ? va : vb));
            const int c = k < 3 ? k : k - 3;
            atomic_add_f32(p + (c == 2 ? 3 : c), s);
        }
        t.has = t.has && !mine;
    }
    if (t.has) {
        float4 *ga = gclip + t.va, *gb = gclip + t.vb;
        atomic_add_f32(&ga->x, t.g[0]);
        atomic_add_f32(&ga->y, t.g[1]);
        atomic_add_f32(&ga->w, t.g[2]);
        atomic_add_f32(&gb->x, t.g[3]);
        atomic_add_f32(&gb->y, t.g[4]);
        atomic_add_f32(&gb->w, t.g[5]);
    }
}

// ----------------------------------------------------------------------------- camera smoothing^T

// A wave per 64 x 4 region for a chunk of the camera's renders: as in the
// forward, the pairs are evaluated once, a pair a lane.  A pair across a
// region's border is evaluated in both; the region of its receiving sample
// adds the edge's terms.  64 512^2 images 188 -> 101 us; a 1920 x 1080 image
// with long outlines 260 -> 30 and a 256^2 one 46 -> 10, where the atomics of
// all samples of an outline met on its two vertices.  One channel at 6 waves
// per SIMD (4: 117 us), three at 4.
template <int C>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(C == 1 ? 6 : 4))) void aa_camera_backward_kernel(
    const ViewConst *__restrict__ views, int L, const RenderConst *__restrict__ renders,
    const int *__restrict__ cam_renders_off, const int *__restrict__ cam_renders, int chunk,
    const TriSetup *__restrict__ setup, const int *__restrict__ faces, const unsigned char *__restrict__ silm,
    const float *__restrict__ verts, const unsigned long long *__restrict__ keys,
    const unsigned char *__restrict__ aa_flag, const float *__restrict__ img0, const float *__restrict__ gimg,
    float *__restrict__ gimg0, float4 *__restrict__ gclip) {
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
    float gself[kAaH][C];
    bool flagged = false;
#pragma unroll
    for (int q = 0; q < kAaH; ++q) {
        const bool live = i < W && j0 + q < H;
        const long long p = (long long)(j0 + q) * W + i;
#pragma unroll
        for (int c = 0; c < C; ++c) gself[q][c] = live ? gimg[base + p * C + c] : 0.f;
        // samples the forward found without candidate pairs pass the gradient through
        flagged = flagged || (live && v.antialias && v.nfaces > 0 && aa_flag[v.pix_off + p]);
    }
    int n = 0;
    if (__ballot(flagged) != 0ull) {
        const unsigned long long *kv = keys + v.pix_off;
        n = aa_list(g, aa_keys(kv, W, H, i0, j0, lane), silm + v.setup_off, lane);
        for (int e0 = 0; e0 < n; e0 += 64) {      // uniform
            const int e = e0 + lane;
            EdgeTerm t;
            t.has = false;
            t.va = t.vb = 0;
            if (e < n) {
                const int slot = g.item[e];
                const AASlot s = aa_slot(slot);
                const long long pa = (long long)(j0 + s.ja) * W + i0 + s.ia, pb = (long long)(j0 + s.jb) * W + i0 + s.ib;
                const unsigned long long ka = kv[pa], kb = kv[pb];
                const bool front = ka < kb;
                AAPair pr{};
                if (aa_eval<true>(v, setup, faces, silm, verts, front ? (unsigned)ka : (unsigned)kb, front, i0 + s.ia,
                                  j0 + s.ja, i0 + s.ib, j0 + s.jb, s.horiz, pr)) {
                    const unsigned char recv = aa_receiver(pr, front);
                    g.state[slot] = kAaCand | recv;
                    g.w[slot] = pr.w;
                    const bool ra = recv == kAaA;
                    if (ra ? aa_inside(s.ia, s.ja) : aa_inside(s.ib, s.jb)) {
                        const long long ps = ra ? pa : pb, pn = ra ? pb : pa;
                        double galpha = 0;
                        for (int r = r0; r < r1; ++r) {
                            const long long b = renders[cam_renders[r]].img_off;
#pragma unroll
                            for (int c = 0; c < C; ++c)
                                galpha += (double)gimg[b + ps * C + c] * (img0[b + pn * C + c] - img0[b + ps * C + c]);
                        }
                        edge_set(t, pr, galpha);
                    }
                }
            }
            edge_add(t, gclip + v.clip_off);
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
            for (int c = 0; c < C; ++c) acc[c] = gself[q][c];
            if (n)
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int slot = aa_slot_of(lane, q, d);
                    const unsigned st = g.state[slot];
                    if (!(st & (kAaA | kAaB))) continue;
                    const float w = g.w[slot];
                    const long long pn = p + (d == 0 ? -1 : d == 1 ? 1 : d == 2 ? -W : W);
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        if (st & aa_self_bit(d)) acc[c] -= w * gself[q][c];
                        else acc[c] += w * gimg[base + pn * C + c];
                }
#pragma unroll
            for (int c = 0; c < C; ++c) gimg0[base + p * C + c] = acc[c];
        }
        if (++r >= r1) break;
        base = renders[cam_renders[r]].img_off;
#pragma unroll
        for (int q = 0; q < kAaH; ++q)
#pragma unroll
            for (int c = 0; c < C; ++c)
                gself[q][c] = i < W && j0 + q < H ? gimg[base + ((long long)(j0 + q) * W + i) * C + c] : 0.f;
    }
}

// ----------------------------------------------------------------------------- reduction by (triangle, tile)

// Float atomics on this GPU are performed at the memory side, so many
// workgroups adding into the same few addresses (the two triangles of a
// ground plane, a light's frame gradient) serialize.  The backward kernels
// therefore avoid hot atomics altogether: they walk the same tiles as the
// rasterizer and, for every triangle binned to a tile, write the sum of that
// triangle's per-pixel gradient terms over the tile's pixels into the
// triangle's slot for that tile (the binning already gave every (triangle,
// tile) pair a unique index).  Later gathers sum those slots per triangle,
// then per vertex (through the vertex -> triangle-corner lists), with plain
// stores.  Per-light terms are written per tile and summed per light the
// same way.  Only triangles that overflowed the bins, the 512-pair items of
// larger triangles, the sparse silhouette terms and the bilinear moment-map
// scatter use atomics, so their sums have no fixed order.
constexpr int kNV = 21;   // per pair: 9 world-position terms, 9 clip (x, y, w) terms, 3 albedo terms

// The rows of pairs (and those of gtri, of triangles that overflowed the bins
// or have many pairs) hold the 21 values as three 8-float corner records,
// [world x y z | clip x y w | albedo term of channel c | pad] for corner c, so
// that the per-vertex gather reads one aligned 32-byte sector per incident
// corner.  row_slot maps value index i to its place in the row.  Rows of light
// views have no albedo terms.
constexpr int kRow = 24;
__host__ __device__ constexpr int row_slot(int i) {
    return i < 9 ? (i / 3) * 8 + i % 3 : i < 18 ? ((i - 9) / 3) * 8 + 3 + (i - 9) % 3 : (i - 18) * 8 + 6;
}
// Value index at place p of a row (pads and, for N < 21, albedo terms repeat value 0).
template <int N>
__host__ __device__ constexpr int row_value(int p) {
    return p % 8 < 3 ? (p / 8) * 3 + p % 8 : p % 8 < 6 ? 9 + (p / 8) * 3 + p % 8 - 3 : p % 8 == 6 && N > 18 ? 18 + p / 8 : 0;
}

template <int T>
struct TileShape {
    static constexpr int NPIX = T * T;
    static constexpr int NT = NPIX < 256 ? NPIX : 256;
    static constexpr int PPT = NPIX / NT;
    static constexpr int NW = NT / 64;
};

// Per-workgroup sum of N per-thread values, written to dst[0..N) by threads < N.  Uniform call.
struct IdentitySlot {
    __device__ int operator()(int i) const { return i; }
};

// Workgroup sums of N values; value i is stored at dst[slot(i)].
template <int NW, int N, class Slot = IdentitySlot>
__device__ __forceinline__ void block_sum_store(const float (&val)[N], float *dst, Slot slot = Slot()) {
    __shared__ float part[NW][32];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    const float t = wave_sum_multi(val);
    const int i = lane >> kSumShift<N>;
    const bool holds = (lane & ((1 << kSumShift<N>) - 1)) == 0 && i < N;
    if (NW == 1) {
        if (holds) dst[slot(i)] = t;
        return;
    }
    if (holds) part[w][i] = t;
    __syncthreads();
    if (threadIdx.x < N) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < NW; ++q) s += part[q][threadIdx.x];
        dst[slot(threadIdx.x)] = s;
    }
}

// For every triangle binned to tile gt: sum of val over the tile's active
// pixels it owns -> pair_sums[pair index][0..N), zeros when it owns none.
// Marks the pixels whose triangle was found.  Uniform call.
//
// The bin is walked in chunks of 64 entries (triangle and pair index, both
// written by the binning pass).  Each pixel finds the entry of its triangle
// (a broadcast LDS scan of the chunk) and adds its N values into that
// entry's LDS row with LDS atomics.  Every entry's pair_flag byte is written
// (1: the row holds a sum, 0: the triangle owns no active pixel here), and
// only flagged rows are stored.  Cost per pixel is N LDS adds however many
// triangles share the tile, so dense meshes (about one triangle per pixel)
// stay cheap.
// The tile's bin range and this thread's entry of its first chunk, loaded
// at the start of a tile kernel so that these dependent loads overlap the
// per-pixel work instead of following it.  Loads are unconditional (clamped
// indices) so that nothing waits for them before their use.
struct BinHead {
    unsigned b0, b1, si, pair;
};
__device__ __forceinline__ BinHead bin_head(int gt, int tid, const unsigned *__restrict__ tile_start,
                                            const unsigned *__restrict__ bins,
                                            const unsigned *__restrict__ bin_pair) {
    BinHead h;
    const int at = gt + (gt >> kScanShift);          // the tile scan keeps an end per kScanBlock tiles
    h.b0 = tile_start[at];
    h.b1 = tile_start[at + 1];
    const unsigned c = h.b1 > h.b0 ? min(h.b0 + (unsigned)tid, h.b1 - 1) : 0u;
    h.si = bins[c];
    h.pair = bin_pair[c];
    return h;
}

template <int T, int N>
__device__ __forceinline__ void tile_pair_sums(const ViewConst &v, const BinHead &head,
                                               const unsigned *__restrict__ bins,
                                               const unsigned *__restrict__ bin_pair,
                                               const int (&key)[TileShape<T>::PPT],
                                               const float (&val)[TileShape<T>::PPT][N],
                                               const bool (&act)[TileShape<T>::PPT],
                                               bool (&matched)[TileShape<T>::PPT],
                                               unsigned char *__restrict__ pair_flag, float *__restrict__ pair_sums) {
    using TS = TileShape<T>;
    constexpr int CH = 64;
    __shared__ float part[CH * N];
    __shared__ __align__(16) int ent[CH];
    __shared__ unsigned slot[CH];
    __shared__ int hit[CH];
    const int tid = threadIdx.x;
    const unsigned b0 = head.b0, b1 = head.b1;
    bool mine = false;
#pragma unroll
    for (int k = 0; k < TS::PPT; ++k) mine = mine || act[k];
    const bool any = __syncthreads_or(mine) != 0;
    for (unsigned c0 = b0; c0 < b1; c0 += CH) {
        const int n = (int)min((unsigned)CH, b1 - c0);
        if (tid < CH) {
            const bool first = c0 == b0;
            // unused entries hold -2, which matches no key (background is -1)
            ent[tid] = tid < n ? (int)((first ? head.si : bins[c0 + tid]) - (unsigned)v.setup_off) : -2;
            slot[tid] = tid < n ? (first ? head.pair : bin_pair[c0 + tid]) : 0u;
            hit[tid] = 0;
        }
        if (any)
            for (int f = tid; f < n * N; f += TS::NT) part[f] = 0.f;
        __syncthreads();
        if (any) {
            int idx[TS::PPT];
#pragma unroll
            for (int k = 0; k < TS::PPT; ++k) idx[k] = -1;
            // fixed-length scan, four entries per LDS read, all reads in flight together
            const int4 *ent4 = reinterpret_cast<const int4 *>(ent);
#pragma unroll
            for (int e4 = 0; e4 < CH / 4; ++e4) {
                const int4 t = ent4[e4];
#pragma unroll
                for (int k = 0; k < TS::PPT; ++k) {
                    idx[k] = key[k] == t.x ? 4 * e4 : idx[k];
                    idx[k] = key[k] == t.y ? 4 * e4 + 1 : idx[k];
                    idx[k] = key[k] == t.z ? 4 * e4 + 2 : idx[k];
                    idx[k] = key[k] == t.w ? 4 * e4 + 3 : idx[k];
                }
            }
            const int lane = tid & 63;
#pragma unroll
            for (int k = 0; k < TS::PPT; ++k) {
                if (idx[k] >= 0) matched[k] = true;
                bool todo = idx[k] >= 0 && act[k];
                // A triangle owning many of the wave's pixels (a large ground
                // polygon) is summed with one multi-value wave reduction; LDS
                // atomics from that many lanes into one row would serialize.
                for (int round = 0; round < 2; ++round) {
                    const unsigned long long m = __ballot(todo);
                    if (m == 0) break;
                    const int leader = __ffsll(m) - 1;
                    const int kk = __builtin_amdgcn_readlane(key[k], leader);
                    const bool in = todo && key[k] == kk;
                    if (__popcll(__ballot(in)) < 16) break;
                    float masked[N];
#pragma unroll
                    for (int i = 0; i < N; ++i) masked[i] = in ? val[k][i] : 0.f;
                    const float t = wave_sum_multi(masked);
                    const int e = __builtin_amdgcn_readlane(idx[k], leader);
                    if ((lane & 1) == 0 && (lane >> 1) < N) atomicAdd(part + e * N + (lane >> 1), t);
                    if (lane == leader) hit[e] = 1;
                    todo = todo && !in;
                }
                if (todo) {
                    hit[idx[k]] = 1;
                    float *row = part + idx[k] * N;
#pragma unroll
                    for (int i = 0; i < N; ++i)
                        if (val[k][i] != 0.f) atomicAdd(row + i, val[k][i]);
                }
            }
            __syncthreads();
        }
        if (tid < n) pair_flag[slot[tid]] = (unsigned char)hit[tid];
        if (any) {
            constexpr int G = 4;                          // LDS reads of G iterations in flight together
            const int iters = (n * N + TS::NT - 1) / TS::NT;
#pragma unroll 1
            for (int it0 = 0; it0 < iters; it0 += G) {
                float pv[G];
                size_t dst[G];
                bool wr[G];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int f = tid + (it0 + g) * TS::NT;
                    const int e = min(f / N, CH - 1), i = f - (f / N) * N;
                    wr[g] = f < n * N && hit[e] != 0;
                    dst[g] = (size_t)slot[e] * kRow + (size_t)row_slot(i);
                    pv[g] = part[min(f, CH * N - 1)];
                }
#pragma unroll
                for (int g = 0; g < G; ++g)
                    if (wr[g]) pair_sums[dst[g]] = pv[g];
            }
        }
        __syncthreads();
    }
}

// Pixels of triangles that overflowed the bins: straight to their rows of gtri.  Uniform call.
template <int PPT, int N>
__device__ __forceinline__ void overflow_rows(const ViewConst &v, const int (&key)[PPT], const float (&val)[PPT][N],
                                              const bool (&active)[PPT], const bool (&matched)[PPT],
                                              float *__restrict__ gtri) {
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const bool a = active[k] && !matched[k];
        if (__ballot(a))
            scatter_by_key(a, key[k], val[k],
                           [&](int t, int i) { return gtri + (size_t)(v.setup_off + t) * kRow + row_slot(i); });
    }
}

// Per-(triangle, tile) sums of one 8x8 tile held by one wave, without walking
// the tile's bin: the pairs of triangle t are the tiles of its bounding box
// in row-major order, numbered from pair_off[t] as the binning numbers them,
// so a pixel finds its row from its triangle's setup record.  Lanes holding
// the same triangle are grouped by a leader loop (one iteration per distinct
// triangle in the wave); a group of 16 or more lanes (a large ground
// polygon) is summed with one multi-value wave reduction, the others with
// LDS atomics into the row of their leader (the group's lowest lane), which
// then stores the row and flags the pair.  The atomics of a group meet on one
// address each, and where the groups are several samples wide that is what
// bounds the sums: horizontal neighbours of one triangle are added first
// (three 2048^2 maps 205 -> 174 us, then 153 with the XCDs in turns; the
// lookup's adjoint at 1080p 120 -> 110, then 81),
// unless few lanes have one (meshes with a sample or two a triangle and tile:
// 187 -> 191 with it).  The test for zero per value is worth its instructions
// (64 scenes 388 us, 465 without it): unlit samples are zero in most values.  Pair flags start at zero (the
// backward clears them), so pairs without a pixel keep flag 0.  Pixels of
// triangles that overflowed the bins stay unmatched for overflow_rows.
// Uniform call (all 64 lanes).
template <int T, int N>
__device__ __forceinline__ void wave_pair_sums(const ViewConst &v, int tx, int ty, int key, const float (&val)[N],
                                               bool act, bool &matched, const TriSetup *__restrict__ setup,
                                               const unsigned *__restrict__ pair_off, unsigned capacity,
                                               unsigned char *__restrict__ pair_flag, float *__restrict__ pair_sums) {
    __shared__ float part[64 * N];
    const int lane = (int)(threadIdx.x & 63);
    unsigned slot = 0;
    bool mine = false;
    // a pixel turned away from its lights has no terms: no sum, and no row for
    // triangles that hold only such pixels (the gather of 64 scenes 51 -> 47 us);
    // light texels that get here have some
    bool some = N <= 18;
#pragma unroll
    for (int i = 0; i < N; ++i) some = some || val[i] != 0.f;
    if (act && some && key >= 0) {
        const int si = v.setup_off + key;
        const unsigned a = pair_off[si], b = pair_off[si + 1];
        if (b <= capacity) {                             // else: the overflow path
            const TriSetup &st = setup[si];
            const int tx0 = st.bx0 / T, ty0 = st.by0 / T, ntx = st.bx1 / T - tx0 + 1;
            slot = a + (unsigned)((ty - ty0) * ntx + (tx - tx0));
            mine = true;
        }
    }
    matched = mine || !some;
    // leader of every lane's group; groups of 16 or more lanes go to the wave reduction
    int leader = lane;
    unsigned long long pending = __ballot(mine), big = 0ull;
    while (pending) {
        const int l = __ffsll(pending) - 1;
        const int kk = __builtin_amdgcn_readlane(key, l);
        const bool in = mine && key == kk;
        const unsigned long long m = __ballot(in);
        pending &= ~m;
        if (in) leader = l;
        if (__popcll(m) >= 16) big |= m;
    }
    while (big) {
        const int l = __ffsll(big) - 1;
        const int kk = __builtin_amdgcn_readlane(key, l);
        const bool in = mine && key == kk;
        big &= ~__ballot(in);
        float masked[N];
#pragma unroll
        for (int i = 0; i < N; ++i) masked[i] = in ? val[i] : 0.f;
        const float t = wave_sum_multi(masked);          // lane 2i: the group's total of value i (17 <= N <= 32)
        const unsigned sl = (unsigned)__builtin_amdgcn_readlane((int)slot, l);
        if ((lane & 1) == 0 && (lane >> 1) < N) pair_sums[(size_t)sl * kRow + row_slot(lane >> 1)] = t;
        if (lane == l) pair_flag[sl] = 1;
        mine = mine && !in;
    }
    const bool lead = mine && leader == lane;
    float sum[N];
    bool own = mine;
    const int beside = dpp_movi<0xB1>(mine ? leader : -1);          // of lane ^ 1, read with every lane active
    const bool same = mine && beside == leader;
    if (__popcll(__ballot(same)) >= 16) {                // uniform
#pragma unroll
        for (int i = 0; i < N; ++i) sum[i] = val[i] + dpp_mov<0xB1>(same ? val[i] : 0.f);
        own = own && !(same && (lane & 1));
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) sum[i] = val[i];
    }
    if (lead) {
#pragma unroll
        for (int i = 0; i < N; ++i) part[lane * N + i] = sum[i];
    }
    __syncthreads();
    if (own && !lead) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (sum[i] != 0.f) atomicAdd(part + leader * N + i, sum[i]);
    }
    __syncthreads();
    if (lead) {
        float4 *row = (float4 *)(pair_sums + (size_t)slot * kRow);
#pragma unroll
        for (int q = 0; q < kRow / 4; ++q)
            row[q] = make_float4(part[lane * N + row_value<N>(4 * q)], part[lane * N + row_value<N>(4 * q + 1)],
                                 part[lane * N + row_value<N>(4 * q + 2)], part[lane * N + row_value<N>(4 * q + 3)]);
        pair_flag[slot] = 1;
    }
    __syncthreads();
}

// ----------------------------------------------------------------------------- lookup^T

// Where one pixel's gradient lands in a light's moment maps: the bilinear
// taps around texel coordinate (ix + fx, iy + fy), weights for (gm1, gm2).
struct MapHit {
    int ix, iy;
    float fx, fy, gm1, gm2;
};

// A camera pixel as its renders share it: the point and normal, recomputed as
// the forward forms them, what the adjoint of those needs, and the gradients
// that every light of every render adds to.  The adjoint from the point and
// the normal to the corners is linear in them, so it runs once per pixel.
struct PixelGeom {
    BaryFull b;
    float px, py;
    float v0[3], v1[3], v2[3], rho[3];
    float x, y, z, nx, ny, nz, rn;
    float gx[3], gn[3];
};

__device__ __forceinline__ void pixel_geom(PixelGeom &g, const ViewConst &cv, const TriVerts &r, int i, int j) {
    g.v0[0] = r.a.x; g.v0[1] = r.a.y; g.v0[2] = r.a.z;
    g.v1[0] = r.a.w; g.v1[1] = r.b.x; g.v1[2] = r.b.y;
    g.v2[0] = r.b.z; g.v2[1] = r.b.w; g.v2[2] = r.c.x;
    g.rho[0] = r.c.y; g.rho[1] = r.c.z; g.rho[2] = r.c.w;          // from the face record
    g.px = ndc_c(i, cv.W);
    g.py = -ndc_c(j, cv.H);
    const float4 c0 = clip_of(cv.M, g.v0[0], g.v0[1], g.v0[2]), c1 = clip_of(cv.M, g.v1[0], g.v1[1], g.v1[2]),
                 c2 = clip_of(cv.M, g.v2[0], g.v2[1], g.v2[2]);
    g.b = bary_full(c0, c1, c2, g.px, g.py);
    g.x = (g.b.b0 * g.v0[0] + g.b.b1 * g.v1[0]) + g.b.b2 * g.v2[0];
    g.y = (g.b.b0 * g.v0[1] + g.b.b1 * g.v1[1]) + g.b.b2 * g.v2[1];
    g.z = (g.b.b0 * g.v0[2] + g.b.b1 * g.v1[2]) + g.b.b2 * g.v2[2];
    const float e1x = g.v1[0] - g.v0[0], e1y = g.v1[1] - g.v0[1], e1z = g.v1[2] - g.v0[2];
    const float e2x = g.v2[0] - g.v0[0], e2y = g.v2[1] - g.v0[1], e2z = g.v2[2] - g.v0[2];
    const float crx = e1y * e2z - e1z * e2y, cry = e1z * e2x - e1x * e2z, crz = e1x * e2y - e1y * e2x;
    g.rn = __builtin_amdgcn_rsqf((crx * crx + cry * cry) + crz * crz);
    g.nx = crx * g.rn;
    g.ny = cry * g.rn;
    g.nz = crz * g.rn;
#pragma unroll
    for (int k = 0; k < 3; ++k) g.gx[k] = g.gn[k] = 0.f;
}

// One light of one render: the shade it adds, its terms in gx and gn, this
// pixel's gradient w.r.t. the light parameter (al) and its map gradient.
__device__ __forceinline__ void light_terms(PixelGeom &g, const ViewConst &l, const float *__restrict__ J,
                                            const float *__restrict__ maps, float srho, float &shade, float (&al)[3],
                                            MapHit &hit) {
    const float x = g.x, y = g.y, z = g.z, nx = g.nx, ny = g.ny, nz = g.nz;
    const float *M = l.M;
    // outside its own directions a cube face adds nothing, nor any gradient
    if (l.kind == kCubeFace && cube_face_of(x - l.pos[0], y - l.pos[1], z - l.pos[2]) != l.cube_face) return;
    const float cx = ((M[0] * x + M[1] * y) + M[2] * z) + M[3];
    const float cy = ((M[4] * x + M[5] * y) + M[6] * z) + M[7];
    const float cw = ((M[12] * x + M[13] * y) + M[14] * z) + M[15];
    const float rcw = __builtin_amdgcn_rcpf(cw);
    const float ux = cx * rcw, uy = cy * rcw;
    const bool inside = cw > 0.f && fabsf(ux) <= 1.f && fabsf(uy) <= 1.f;
    float vis = 1.f, visr = 1.f, zz = 0.f, zw = 0.f, floor_v = 0.f, m1 = 0.f, m2 = 0.f, var = 0.f, dd = 0.f, fx = 0.f,
          fy = 0.f;
    int ixs = 0, iys = 0;
    // the direction to the light, with one distance for the receiver depth, the
    // shading and their adjoints (the correctly rounded root is 16 instructions)
    const bool directional = l.kind == kDirectional;
    float ox, oy, oz, olen = 1.f, rol = 1.f;
    if (directional) {
        ox = -l.dir[0]; oy = -l.dir[1]; oz = -l.dir[2];
    } else {
        ox = l.pos[0] - x; oy = l.pos[1] - y; oz = l.pos[2] - z;
        olen = sqrtf((ox * ox + oy * oy) + oz * oz);
        rol = grcp(olen);
        ox *= rol; oy *= rol; oz *= rol;
    }
    const int S = l.W;
    // filtered maps are stored with side Sp; cube faces keep P texels of
    // their neighbours around the face, so taps may cross the seam
    const int P = l.fpad, Sp = S + 2 * P;
    // filtered maps hold (m1, m2) interleaved per texel
    const float2 *mm = (const float2 *)(maps + l.fmap_off);
    float2 t00 = make_float2(0.f, 0.f), t01 = t00, t10 = t00, t11 = t00;
    if (inside) {
        const float sx = (ux + 1.f) * (0.5f * S) - 0.5f;
        const float sy = (1.f - uy) * (0.5f * S) - 0.5f;
        const float fx0 = floorf(sx), fy0 = floorf(sy);
        fx = sx - fx0;
        fy = sy - fy0;
        const int ix = (int)fx0 + P, iy = (int)fy0 + P;
        ixs = ix;
        iys = iy;
        const int x0 = min(max(ix, 0), Sp - 1), x1 = min(max(ix + 1, 0), Sp - 1);
        const int y0 = min(max(iy, 0), Sp - 1), y1 = min(max(iy + 1, 0), Sp - 1);
        const float w00 = (1.f - fx) * (1.f - fy), w01 = fx * (1.f - fy), w10 = (1.f - fx) * fy, w11 = fx * fy;
        t00 = mm[y0 * Sp + x0]; t01 = mm[y0 * Sp + x1]; t10 = mm[y1 * Sp + x0]; t11 = mm[y1 * Sp + x1];
        m1 = ((w00 * t00.x + w01 * t01.x) + w10 * t10.x) + w11 * t11.x;
        m2 = ((w00 * t00.y + w01 * t01.y) + w10 * t10.y) + w11 * t11.y;
        const float depth =
            directional ? ((x - l.pos[0]) * l.dir[0] + (y - l.pos[1]) * l.dir[1]) + (z - l.pos[2]) * l.dir[2] : olen;
        zz = depth * grcp(l.zfar) - l.zc;
        warp_receiver(l, zz, zw, floor_v);
        var = fmaxf(m2 - m1 * m1, floor_v);
        dd = zw - m1;
        visr = (zw <= m1) ? 1.f : var * grcp(var + dd * dd);
        vis = bleed_reduce(l, visr);
    }
    const float ndo = (nx * ox + ny * oy) + nz * oz;
    const float lam = fmaxf(ndo, 0.f);
    float cone = 1.f;
    if (l.kind == kSpot) {
        const float ca = -((ox * l.dir[0] + oy * l.dir[1]) + oz * l.dir[2]);
        cone = ca >= l.cos_half ? 1.f : 0.f;
    }
    shade += lam * vis * l.intensity * cone;
    const float gvis = srho * lam * l.intensity * cone;
    const float glam = srho * vis * l.intensity * cone;
    const float gndo = ndo > 0.f ? glam : 0.f;
    // from here on only gradient terms are formed: fused multiply-adds
    // (nothing below feeds a forward value or a decision)
    g.gn[0] = fmaf(gndo, ox, g.gn[0]); g.gn[1] = fmaf(gndo, oy, g.gn[1]); g.gn[2] = fmaf(gndo, oz, g.gn[2]);
    const float gox = gndo * nx, goy = gndo * ny, goz = gndo * nz;
    // this pixel's gradient w.r.t. the light frame (M, pos, dir), pulled
    // back to the light parameter through the frame's Jacobian at the end
    float gpos[3] = {0.f, 0.f, 0.f}, gdir[3] = {0.f, 0.f, 0.f};
    float gcx = 0.f, gcy = 0.f, gcw = 0.f;
    if (l.kind == kDirectional) {
        gdir[0] -= gox; gdir[1] -= goy; gdir[2] -= goz;
    } else {
        const float od = fmaf(oz, goz, fmaf(oy, goy, ox * gox));
        const float gpx = fmaf(-ox, od, gox) * rol, gpy = fmaf(-oy, od, goy) * rol, gpz = fmaf(-oz, od, goz) * rol;
        gpos[0] += gpx; gpos[1] += gpy; gpos[2] += gpz;
        g.gx[0] -= gpx; g.gx[1] -= gpy; g.gx[2] -= gpz;
    }
    // through the bleeding reduction: slope 1 / (1 - a) on [a, 1], else 0
    const float gvr = l.bleed > 0.f ? (visr >= l.bleed ? gvis / (1.f - l.bleed) : 0.f) : gvis;
    if (inside && gvr != 0.f && zw > m1) {
        const float qd = var + dd * dd;
        float dv_dmu, dv_dvar_raw;
        if (l.warp_c > 0.f) {
            // exponential maps: the squares of var and dd overflow float32
            const float rq = grcp(qd);
            const float tv = var * rq, td = dd * rq;
            dv_dmu = 2.f * tv * td;
            dv_dvar_raw = td * td;
        } else {
            const float rq2 = grcp(qd * qd);
            dv_dmu = 2.f * var * dd * rq2;
            dv_dvar_raw = dd * dd * rq2;
        }
        const bool clamped = m2 - m1 * m1 < floor_v;
        const float dv_dvar = clamped ? 0.f : dv_dvar_raw;
        const float gm1 = gvr * fmaf(-2.f * m1, dv_dvar, dv_dmu);
        const float gm2 = gvr * dv_dvar;
        // d v / d (receiver depth): through d - mu, through the floor when
        // it binds and follows the warp, and through the warp itself
        float dv_dzw = -dv_dmu;
        if (l.warp_c > 0.f) {
            if (clamped) dv_dzw = fmaf(dv_dvar_raw, 2.f * l.min_var * l.warp_c * l.warp_c * zw, dv_dzw);
            dv_dzw *= l.warp_c * zw;
        }
        const float gdepth = gvr * dv_dzw * grcp(l.zfar);
        if (l.kind == kDirectional) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                g.gx[k] = fmaf(gdepth, l.dir[k], g.gx[k]);
                gpos[k] = fmaf(-gdepth, l.dir[k], gpos[k]);
            }
            gdir[0] = fmaf(gdepth, x - l.pos[0], gdir[0]);
            gdir[1] = fmaf(gdepth, y - l.pos[1], gdir[1]);
            gdir[2] = fmaf(gdepth, z - l.pos[2], gdir[2]);
        } else {
            g.gx[0] = fmaf(-gdepth, ox, g.gx[0]); g.gx[1] = fmaf(-gdepth, oy, g.gx[1]);
            g.gx[2] = fmaf(-gdepth, oz, g.gx[2]);
            gpos[0] = fmaf(gdepth, ox, gpos[0]); gpos[1] = fmaf(gdepth, oy, gpos[1]);
            gpos[2] = fmaf(gdepth, oz, gpos[2]);
        }
        hit = MapHit{ixs, iys, fx, fy, gm1, gm2};        // bilinear scatter to the moment maps
        // the map position moves with x and with the light camera
        // d m / d(fx, fy): each a lerp of two texel differences
        const float a1 = t01.x - t00.x, b1 = t11.x - t10.x, c1 = t10.x - t00.x, d1 = t11.x - t01.x;
        const float a2 = t01.y - t00.y, b2 = t11.y - t10.y, c2 = t10.y - t00.y, d2 = t11.y - t01.y;
        const float dm1fx = fmaf(fy, b1 - a1, a1), dm1fy = fmaf(fx, d1 - c1, c1);
        const float dm2fx = fmaf(fy, b2 - a2, a2), dm2fy = fmaf(fx, d2 - c2, c2);
        const float hs = 0.5f * S;
        const float gsx = fmaf(gm2, dm2fx, gm1 * dm1fx) * hs;
        const float gsy = fmaf(gm2, dm2fy, gm1 * dm1fy) * hs;
        gcx = gsx * rcw;
        gcy = -gsy * rcw;
        gcw = fmaf(-gsx, cx, gsy * cy) * (rcw * rcw);
#pragma unroll
        for (int k = 0; k < 3; ++k) g.gx[k] = fmaf(M[12 + k], gcw, fmaf(M[4 + k], gcy, fmaf(M[k], gcx, g.gx[k])));
    }
    // dL/dM = (gcx, gcy, 0, gcw) outer [x, 1]; with dL/dpos, dL/ddir through J
    const float xh[4] = {x, y, z, 1.f};
    // per parameter j: sum over rows r in (x, y, w) of g_r (J_r(j) . [x, 1]),
    // plus the position and direction terms
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        float u[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int row = r == 0 ? 0 : r == 1 ? 4 : 12;
            u[r] = fmaf(xh[2], J[3 * (row + 2) + j],
                        fmaf(xh[1], J[3 * (row + 1) + j], fmaf(xh[0], J[3 * row + j], J[3 * (row + 3) + j])));
        }
        float a = fmaf(gcw, u[2], fmaf(gcy, u[1], fmaf(gcx, u[0], al[j])));
#pragma unroll
        for (int i = 0; i < 3; ++i) a = fmaf(gpos[i], J[3 * (16 + i) + j], a);
        if (directional)
#pragma unroll
            for (int i = 0; i < 3; ++i) a = fmaf(gdir[i], J[3 * (19 + i) + j], a);
        al[j] = a;
    }
}

// From the point and the normal to the corners: vals[0..9) the corners' world
// positions, vals[9..18) their clip (x, y, w).
__device__ __forceinline__ void pixel_adjoint(const PixelGeom &g, float (&vals)[kNV]) {
    const float e1x = g.v1[0] - g.v0[0], e1y = g.v1[1] - g.v0[1], e1z = g.v1[2] - g.v0[2];
    const float e2x = g.v2[0] - g.v0[0], e2y = g.v2[1] - g.v0[1], e2z = g.v2[2] - g.v0[2];
    // normal: n = cr / |cr|, cr = e1 x e2
    const float ndg = fmaf(g.nz, g.gn[2], fmaf(g.ny, g.gn[1], g.nx * g.gn[0]));
    const float gcr[3] = {fmaf(-g.nx, ndg, g.gn[0]) * g.rn, fmaf(-g.ny, ndg, g.gn[1]) * g.rn,
                          fmaf(-g.nz, ndg, g.gn[2]) * g.rn};
    const float ge1[3] = {fmaf(e2y, gcr[2], -e2z * gcr[1]), fmaf(e2z, gcr[0], -e2x * gcr[2]),
                          fmaf(e2x, gcr[1], -e2y * gcr[0])};
    const float ge2[3] = {fmaf(gcr[1], e1z, -gcr[2] * e1y), fmaf(gcr[2], e1x, -gcr[0] * e1z),
                          fmaf(gcr[0], e1y, -gcr[1] * e1x)};
    // x = sum b_i v_i
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        vals[k] = fmaf(g.b.b0, g.gx[k], -ge1[k]) - ge2[k];
        vals[3 + k] = fmaf(g.b.b1, g.gx[k], ge1[k]);
        vals[6 + k] = fmaf(g.b.b2, g.gx[k], ge2[k]);
    }
    const float gb0 = fmaf(g.gx[2], g.v0[2], fmaf(g.gx[1], g.v0[1], g.gx[0] * g.v0[0]));
    const float gb1 = fmaf(g.gx[2], g.v1[2], fmaf(g.gx[1], g.v1[1], g.gx[0] * g.v1[0]));
    const float gb2 = fmaf(g.gx[2], g.v2[2], fmaf(g.gx[1], g.v2[1], g.gx[0] * g.v2[0]));
    float gc[9];
    bary_backward(g.b, g.px, g.py, gb0, gb1, gb2, gc);
#pragma unroll
    for (int k = 0; k < 9; ++k) vals[9 + k] = gc[k];
}

// Bilinear scatter of one light's moment-map gradient from the pixels of a
// tile.  Each wave adds its taps into an LDS window of WIN x WIN texels
// anchored at the smallest tap it touches, then adds the non-zero values of
// the texels its taps can reach (the taps' bounding box, clipped to the
// window) to global memory: lit pixels carry no map gradient, so most
// windows hold a few texels, not WIN x WIN.  Taps outside the window go to
// global memory directly.  Uniform call.
template <int NW, int PPT, int WIN>
__device__ __forceinline__ void map_window_scatter(const MapHit (&hit)[PPT], int S, float *__restrict__ gmap) {
    static_assert(WIN == 16 || WIN == 32, "the window's rows are walked in powers of two");
    __shared__ float2 win[NW][WIN * WIN];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // smallest and largest tap, (x, y) packed in 16 bits each (S is at most 8192 and its padding)
    unsigned lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int k = 0; k < PPT; ++k)
        if (hit[k].gm1 != 0.f || hit[k].gm2 != 0.f) {
            lo = pk_best<false>(lo, (unsigned)min(max(hit[k].ix, 0), S - 1) | (unsigned)min(max(hit[k].iy, 0), S - 1) << 16);
            hi = pk_best<true>(hi, (unsigned)min(max(hit[k].ix + 1, 0), S - 1) |
                                       (unsigned)min(max(hit[k].iy + 1, 0), S - 1) << 16);
        }
    lo = wave_pk_best<false>(lo);
    const bool any = lo != 0xFFFFFFFFu;
    if (NW == 1 && !any) return;
    hi = wave_pk_best<true>(hi);
    const int mx = (int)(lo & 0xFFFFu), my = (int)(lo >> 16);
    // every tap that lands in the window lies in the bounding box
    const int bw = any ? min((int)(hi & 0xFFFFu) - mx + 1, WIN) : 0, bh = any ? min((int)(hi >> 16) - my + 1, WIN) : 0;
    // lanes over the box: 8 columns wide where that holds it
    const int cs = bw <= 8 ? 3 : WIN == 16 ? 4 : 5, ex = lane & ((1 << cs) - 1), ey0 = lane >> cs, es = 64 >> cs;
    if (ex < bw)
        for (int ey = ey0; ey < bh; ey += es) win[w][ey * WIN + ex] = make_float2(0.f, 0.f);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const MapHit &h = hit[k];
        if (h.gm1 == 0.f && h.gm2 == 0.f) continue;
        const int x0 = min(max(h.ix, 0), S - 1), x1 = min(max(h.ix + 1, 0), S - 1);
        const int y0 = min(max(h.iy, 0), S - 1), y1 = min(max(h.iy + 1, 0), S - 1);
        const float w00 = (1.f - h.fx) * (1.f - h.fy), w01 = h.fx * (1.f - h.fy);
        const float w10 = (1.f - h.fx) * h.fy, w11 = h.fx * h.fy;
        if (x1 - mx < WIN && y1 - my < WIN) {
            float2 *o = win[w] + (y0 - my) * WIN + (x0 - mx);
            const int dx = x1 - x0, dy = (y1 - y0) * WIN;
            atomicAdd(&o[0].x, h.gm1 * w00); atomicAdd(&o[dx].x, h.gm1 * w01);
            atomicAdd(&o[dy].x, h.gm1 * w10); atomicAdd(&o[dy + dx].x, h.gm1 * w11);
            atomicAdd(&o[0].y, h.gm2 * w00); atomicAdd(&o[dx].y, h.gm2 * w01);
            atomicAdd(&o[dy].y, h.gm2 * w10); atomicAdd(&o[dy + dx].y, h.gm2 * w11);
        } else {
            float *a = gmap, *b = gmap + 1;          // interleaved (m1, m2): texel o at 2 o
            const long long o00 = 2 * ((long long)y0 * S + x0), o01 = 2 * ((long long)y0 * S + x1);
            const long long o10 = 2 * ((long long)y1 * S + x0), o11 = 2 * ((long long)y1 * S + x1);
            atomic_add_f32(a + o00, h.gm1 * w00); atomic_add_f32(a + o01, h.gm1 * w01);
            atomic_add_f32(a + o10, h.gm1 * w10); atomic_add_f32(a + o11, h.gm1 * w11);
            atomic_add_f32(b + o00, h.gm2 * w00); atomic_add_f32(b + o01, h.gm2 * w01);
            atomic_add_f32(b + o10, h.gm2 * w10); atomic_add_f32(b + o11, h.gm2 * w11);
        }
    }
    __syncthreads();
    if (ex < bw)
        for (int ey = ey0; ey < bh; ey += es) {
            const float2 t = win[w][ey * WIN + ex];
            float *o = gmap + 2 * ((long long)(my + ey) * S + (mx + ex));
            if (t.x != 0.f) atomic_add_f32(o, t.x);
            if (t.y != 0.f) atomic_add_f32(o + 1, t.y);
        }
    __syncthreads();
}

// Per camera tile, for every render of the camera and every light of the
// render in turn: the light's terms of each pixel, their map gradient through
// the LDS window, the tile's share of the light-parameter gradient; then once
// per pixel the adjoint to the corners and the per-(triangle, tile) sums.
// Nothing is kept per light, so the registers do not depend on how many there
// are (arrays over 4 or 16 lights spilled, and 16 scattered with global
// atomics), and a camera's renders share the point, the normal and their
// adjoint.  Vector issue bounds it, then the latency of key -> record -> taps.
// 64 renders with a light each 494 -> 388 us (5 waves per SIMD; 4: 5% more), 16
// cameras with 8 renders each 716 -> 477, a 1080p RGB render with 3 lights
// 205 -> 81 (4 waves; 5: 3% more).
template <int T, int C>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(T == 32 ? 2 : C == 1 ? 5 : 4))) void lookup_backward_kernel(
    const ViewConst *__restrict__ views, int L, const RenderConst *__restrict__ renders,
    const int *__restrict__ cam_renders_off, const int *__restrict__ cam_renders,
    const int *__restrict__ render_lights, const TriVerts *__restrict__ tv, const unsigned long long *__restrict__ keys,
    const float *__restrict__ maps, const float *__restrict__ gimg0, float *__restrict__ gmaps,
    const TriSetup *__restrict__ setup, const unsigned *__restrict__ tile_start, const unsigned *__restrict__ bins,
    const unsigned *__restrict__ bin_pair, unsigned char *__restrict__ pair_flag, float *__restrict__ pair_sums,
    float *__restrict__ gtri, float *__restrict__ part_render, const float *__restrict__ jac,
    const unsigned *__restrict__ pair_off, unsigned capacity) {
    using TS = TileShape<T>;
    // one wave per 8x8 tile: pair rows found from the setup records (wave_pair_sums)
    constexpr bool kWavePairs = T == 8;
    const Blk blk = xcd_block2<128, 4096>();
    const int cam = blk.y;
    const ViewConst &cv = views[L + cam];
    const int lt = blk.x;
    if (lt >= cv.tiles_x * cv.tiles_y) return;     // whole workgroup
    const int gt = cv.tile_off + lt;
    BinHead head{};
    if (!kWavePairs) head = bin_head(gt, (int)threadIdx.x, tile_start, bins, bin_pair);
    const int tx = lt % cv.tiles_x, ty = lt / cv.tiles_x;
    const int tid = threadIdx.x;
    const int rr0 = cam_renders_off[cam], rr1 = cam_renders_off[cam + 1];
    int key[TS::PPT], pp[TS::PPT];
    bool act[TS::PPT], matched[TS::PPT];
    PixelGeom geo[TS::PPT];
    float galb[TS::PPT][3];
    const float *gfirst = gimg0 + (rr0 < rr1 ? renders[cam_renders[rr0]].img_off : 0);
    float g0[TS::PPT][C];        // upstream gradient in the first render, requested with the keys
#pragma unroll
    for (int k = 0; k < TS::PPT; ++k) {
        const int l = tid + k * TS::NT;
        const int i = tx * T + (l % T), j = ty * T + (l / T);
        const bool in = i < cv.W && j < cv.H;
        pp[k] = in ? j * cv.W + i : 0;
        const unsigned long long kk = in ? keys[cv.pix_off + pp[k]] : kBgKey;
        key[k] = kk == kBgKey ? -1 : (int)(unsigned)kk;
#pragma unroll
        for (int c = 0; c < C; ++c) g0[k][c] = rr0 < rr1 ? gfirst[(long long)pp[k] * C + c] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < TS::PPT; ++k) {
        act[k] = false;
        matched[k] = false;
        galb[k][0] = galb[k][1] = galb[k][2] = 0.f;
        if (key[k] >= 0) {
            const int l = tid + k * TS::NT;
            pixel_geom(geo[k], cv, tv[cv.face_off + key[k]], tx * T + (l % T), ty * T + (l / T));
        }
    }
    for (int rr = rr0; rr < rr1; ++rr) {
        const RenderConst &R = renders[cam_renders[rr]];
        float g[TS::PPT][C], srho[TS::PPT], shade[TS::PPT];
        bool on[TS::PPT];
#pragma unroll
        for (int k = 0; k < TS::PPT; ++k) {
            on[k] = false;
            srho[k] = shade[k] = 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                g[k][c] = rr == rr0 ? g0[k][c] : gimg0[R.img_off + (long long)pp[k] * C + c];
                on[k] = on[k] || g[k][c] != 0.f;
            }
            on[k] = on[k] && key[k] >= 0;
            act[k] = act[k] || on[k];
            if (on[k])
#pragma unroll
                for (int c = 0; c < C; ++c) srho[k] += g[k][c] * geo[k].rho[c];
        }
        const int ntiles = cv.tiles_x * cv.tiles_y;
        for (int q = 0; q < R.light_count; ++q) {
            const int li = render_lights[R.light_begin + q];
            const ViewConst &l = views[li];
            float al[3] = {0.f, 0.f, 0.f};
            MapHit hits[TS::PPT];
#pragma unroll
            for (int k = 0; k < TS::PPT; ++k) {
                hits[k] = MapHit{0, 0, 0.f, 0.f, 0.f, 0.f};
                if (on[k]) light_terms(geo[k], l, jac + (size_t)kJac * li, maps, srho[k], shade[k], al, hits[k]);
            }
            map_window_scatter<TS::NW, TS::PPT, (T == 32 ? 32 : 16)>(hits, l.W + 2 * l.fpad, gmaps + l.fmap_off);
            block_sum_store<TS::NW>(al, part_render + R.part_off + ((long long)q * ntiles + lt) * 3);
        }
#pragma unroll
        for (int k = 0; k < TS::PPT; ++k)
            if (on[k])
#pragma unroll
                for (int c = 0; c < C; ++c) galb[k][c] += g[k][c] * shade[k];
    }
    float val[TS::PPT][kNV];
#pragma unroll
    for (int k = 0; k < TS::PPT; ++k) {
#pragma unroll
        for (int i = 0; i < kNV; ++i) val[k][i] = 0.f;
        if (!act[k]) continue;
        pixel_adjoint(geo[k], val[k]);
#pragma unroll
        for (int c = 0; c < C; ++c) val[k][18 + c] = galb[k][c];
    }
    if constexpr (kWavePairs)
        wave_pair_sums<T, kNV>(cv, tx, ty, key[0], val[0], act[0], matched[0], setup, pair_off, capacity, pair_flag,
                               pair_sums);
    else
        tile_pair_sums<T, kNV>(cv, head, bins, bin_pair, key, val, act, matched, pair_flag, pair_sums);
    overflow_rows(cv, key, val, act, matched, gtri);
}

// ----------------------------------------------------------------------------- light smoothing^T + resolve^T

template <int T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void light_backward_kernel(
    const ViewConst *__restrict__ views, const TriSetup *__restrict__ setup, const int *__restrict__ faces,
    const unsigned char *__restrict__ silm, const float *__restrict__ verts, const TriVerts *__restrict__ tv,
    const unsigned long long *__restrict__ keys, const unsigned char *__restrict__ aa_flag,
    const float *__restrict__ F0, const float *__restrict__ gF1, float4 *__restrict__ gclip, const unsigned *__restrict__ tile_start, const unsigned *__restrict__ bins,
    const unsigned *__restrict__ bin_pair, unsigned char *__restrict__ pair_flag, float *__restrict__ pair_sums,
    float *__restrict__ gtri, float *__restrict__ part_light, const float *__restrict__ jac,
    const unsigned *__restrict__ pair_off, unsigned capacity) {
    using TS = TileShape<T>;
    // one wave per 8x8 tile: pair rows found from the setup records (wave_pair_sums)
    constexpr bool kWavePairs = T == 8;
    const Blk blk = xcd_block2<128, 4096>();
    const int lidx = blk.y;
    const ViewConst &l = views[lidx];
    const int S = l.W;
    const long long plane = (long long)S * S;
    const int lt = blk.x;
    if (lt >= l.tiles_x * l.tiles_y) return;     // whole workgroup
    const int gt = l.tile_off + lt;
    BinHead head{};
    if (!kWavePairs) head = bin_head(gt, (int)threadIdx.x, tile_start, bins, bin_pair);
    const int tx = lt % l.tiles_x, ty = lt / l.tiles_x;
    const unsigned long long *kv = keys + l.pix_off;
    const float *f0a = F0 + l.map_off / 2;      // f; f^2 is its square
    const float *ga = gF1 + l.map_off, *gbp = gF1 + l.map_off + plane;
    __shared__ AAPairs<TS::NT> pairs;
    float accl[6] = {0, 0, 0, 0, 0, 0};
    int key[TS::PPT];
    bool act[TS::PPT], matched[TS::PPT];
    float val[TS::PPT][18];
#pragma unroll
    for (int k = 0; k < TS::PPT; ++k) {
        const int lix = threadIdx.x + k * TS::NT;
        const int i = tx * T + (lix % T), j = ty * T + (lix / T);
        const bool in = i < S && j < S;
        const int pp = in ? j * S + i : 0;
        const unsigned long long ks = kv[pp];
        key[k] = (in && ks != kBgKey) ? (int)(unsigned)ks : -1;
        matched[k] = false;
#pragma unroll
        for (int q = 0; q < 18; ++q) val[k][q] = 0.f;
        float g0 = in ? ga[pp] : 0.f, g1 = in ? gbp[pp] : 0.f;
        if (l.antialias && l.nfaces > 0) {                       // uniform
            bool cand[4] = {false, false, false, false};
            // texels the forward found without candidate pairs skip the smoothing terms
            const bool flagged = in && aa_flag[l.pix_off + pp];
            const int tid = (int)threadIdx.x;
            unsigned n = 0;
            if (TS::NW > 1 || __ballot(flagged) != 0ull) {
                if (flagged) aa_candidates(l, kv, silm, ks, i, j, cand);
                if (k > 0) __syncthreads();
                aa_pairs_list(pairs, tid, cand);
                __syncthreads();
                n = aa_pairs_total(pairs);
                for (unsigned e0 = (unsigned)(tid & ~63); e0 < n; e0 += TS::NT) {      // uniform in the wave
                    const unsigned e = e0 + (unsigned)(tid & 63);
                    EdgeTerm t;
                    t.has = false;
                    t.va = t.vb = 0;
                    if (e < n) {
                        const unsigned slot = aa_pairs_item(pairs, e);
                        const int d = slot & 3, u = (int)(slot >> 2) + k * TS::NT;
                        const int is = tx * T + (u % T), js = ty * T + (u / T);
                        const int in_ = is + (d == 0 ? -1 : d == 1 ? 1 : 0), jn = js + (d == 2 ? -1 : d == 3 ? 1 : 0);
                        const int ps = js * S + is, pn = jn * S + in_;
                        const unsigned long long kp = kv[ps], kn = kv[pn];
                        const float fs0 = f0a[ps], fs1 = fs0 * fs0, fn0 = f0a[pn], fn1 = fn0 * fn0, gs0 = ga[ps],
                                    gs1 = gbp[ps];
                        const bool front = kp < kn;
                        AAPair pr{};
                        const bool ok = aa_eval<true>(l, setup, faces, silm, verts, front ? (unsigned)kp : (unsigned)kn,
                                                      front, is, js, in_, jn, d < 2, pr);
                        const bool self_recv = (pr.recv == 1) != front;
                        pairs.state[slot] = !ok ? 0 : self_recv ? 1 : 2;
                        pairs.w[slot] = pr.w;
                        if (ok && self_recv) edge_set(t, pr, (double)gs0 * (fn0 - fs0) + (double)gs1 * (fn1 - fs1));
                    }
                    edge_add(t, gclip + l.clip_off);
                }
            }
            if (n) {
                __syncthreads();
                const float gs0 = g0, gs1 = g1;
                const int q[4] = {pp - 1, pp + 1, pp - S, pp + S};
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    if (!cand[d]) continue;
                    const int st = pairs.state[tid << 2 | d];
                    const float w = pairs.w[tid << 2 | d];
                    if (st == 1) {
                        g0 -= w * gs0;
                        g1 -= w * gs1;
                    } else if (st == 2) {
                        g0 += w * ga[q[d]];
                        g1 += w * gbp[q[d]];
                    }
                }
            }
        }
        // resolve^T: F0 = (z, z^2), z = d(x) / far
        act[k] = key[k] >= 0 && (g0 != 0.f || g1 != 0.f);
        if (act[k]) {
            const TriVerts r = tv[l.face_off + key[k]];
            const float v0[3] = {r.a.x, r.a.y, r.a.z}, v1[3] = {r.a.w, r.b.x, r.b.y}, v2[3] = {r.b.z, r.b.w, r.c.x};
            const float4 c0 = clip_of(l.M, v0[0], v0[1], v0[2]), c1 = clip_of(l.M, v1[0], v1[1], v1[2]),
                         c2 = clip_of(l.M, v2[0], v2[1], v2[2]);
            const float px = ndc_c(i, S), py = -ndc_c(j, S);
            const BaryFull b = bary_full(c0, c1, c2, px, py);
            const float x = (b.b0 * v0[0] + b.b1 * v1[0]) + b.b2 * v2[0];
            const float y = (b.b0 * v0[1] + b.b1 * v1[1]) + b.b2 * v2[1];
            const float z = (b.b0 * v0[2] + b.b1 * v1[2]) + b.b2 * v2[2];
            // F0 = (f, f^2), f = z, or exp(c z) for exponential maps
            const float gz = l.warp_c > 0.f ? l.warp_c * f0a[pp] * (g0 + 2.f * f0a[pp] * g1) : g0 + 2.f * f0a[pp] * g1;
            const float gdepth = gz * grcp(l.zfar);
            float gx[3];
            if (l.kind == kDirectional) {
                gx[0] = gdepth * l.dir[0]; gx[1] = gdepth * l.dir[1]; gx[2] = gdepth * l.dir[2];
                accl[0] -= gx[0]; accl[1] -= gx[1]; accl[2] -= gx[2];
                accl[3] += gdepth * (x - l.pos[0]); accl[4] += gdepth * (y - l.pos[1]); accl[5] += gdepth * (z - l.pos[2]);
            } else {
                const float ddx = x - l.pos[0], ddy = y - l.pos[1], ddz = z - l.pos[2];
                const float dl = sqrtf((ddx * ddx + ddy * ddy) + ddz * ddz);
                const float inv = gdepth * grcp(dl);
                gx[0] = ddx * inv; gx[1] = ddy * inv; gx[2] = ddz * inv;
                accl[0] -= gx[0]; accl[1] -= gx[1]; accl[2] -= gx[2];
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                val[k][q] = b.b0 * gx[q];
                val[k][3 + q] = b.b1 * gx[q];
                val[k][6 + q] = b.b2 * gx[q];
            }
            const float gb0 = (gx[0] * v0[0] + gx[1] * v0[1]) + gx[2] * v0[2];
            const float gb1 = (gx[0] * v1[0] + gx[1] * v1[1]) + gx[2] * v1[2];
            const float gb2 = (gx[0] * v2[0] + gx[1] * v2[1]) + gx[2] * v2[2];
            float gc[9];
            bary_backward(b, px, py, gb0, gb1, gb2, gc);
#pragma unroll
            for (int q = 0; q < 9; ++q) val[k][9 + q] = gc[q];
        }
    }
    // (pos, dir) terms pulled back to the light parameter
    const float *J = jac + (size_t)kJac * lidx;
    float gpar[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < 3; ++i) a += accl[i] * J[3 * (16 + i) + j] + accl[3 + i] * J[3 * (19 + i) + j];
        gpar[j] = a;
    }
    block_sum_store<TS::NW>(gpar, part_light + ((long long)l.part_off + lt) * 3);
    if constexpr (kWavePairs)
        wave_pair_sums<T, 18>(l, tx, ty, key[0], val[0], act[0], matched[0], setup, pair_off, capacity, pair_flag,
                              pair_sums);
    else
        tile_pair_sums<T, 18>(l, head, bins, bin_pair, key, val, act, matched, pair_flag, pair_sums);
    overflow_rows(l, key, val, act, matched, gtri);
}

// ----------------------------------------------------------------------------- gathers

// A triangle's gradient is the sum of its flagged pair rows: up to kOwnRows of
// them are read where it is needed; overflowed triangles and those with more
// pairs have one row in gtri.
struct TriRows {
    const float *rows;       // first row
    unsigned mask;           // rows that hold a sum
};
__device__ __forceinline__ unsigned flag_word(const unsigned char *p) {      // four flag bytes, any alignment
    unsigned w;
    __builtin_memcpy(&w, p, 4);
    return w;
}
// Rows of triangle t with pairs [a, b); w: the flag bytes from a on.
__device__ __forceinline__ TriRows tri_rows(unsigned t, unsigned a, unsigned b, unsigned w, unsigned capacity,
                                            const float *__restrict__ pair_sums, const float *__restrict__ gtri) {
    static_assert(kOwnRows == 4, "one word of flags");
    const unsigned n = b - a;
    // with both ends at kPairEnd it may have pairs or none, and its row is cleared in any case
    if (n > kOwnRows || b > capacity) return TriRows{gtri + (size_t)t * kRow, n || a == kPairEnd ? 1u : 0u};
    const unsigned m = (w & 1u) | (w >> 7 & 2u) | (w >> 14 & 4u) | (w >> 21 & 8u);
    return TriRows{pair_sums + (size_t)a * kRow, m & ((1u << n) - 1u)};
}

// Share blk of kGlightBlocks of the partials that light l's tiles and the tiles of
// each render that uses it left; a few lights with many of them still fill the
// GPU.  A render's tiles are cut only as far as that takes: the way to them
// (render, camera) is a chain of loads, and 16 renders one after the other
// took 20 us.
__device__ __forceinline__ void light_partials(int l, int blk, const ViewConst *__restrict__ views,
                                               const LightSum &ls) {
    const ViewConst &v = views[l];
    float acc[3] = {0.f, 0.f, 0.f};
    const int nlt = v.tiles_x * v.tiles_y;
#pragma unroll 4
    for (int q = blk * 256 + (int)threadIdx.x; q < nlt; q += kGlightBlocks * 256)
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[k] += ls.part_light[((long long)v.part_off + q) * 3 + k];
    const int e0 = ls.light_renders_off[l], n = ls.light_renders_off[l + 1] - e0;
    const int cut = n > 0 ? (kGlightBlocks + n - 1) / n : 1;
    for (int u = blk; u < n * cut; u += kGlightBlocks) {
        const int e = ls.light_renders[e0 + u / cut], r = e >> 5, slot = e & 31;
        const RenderConst &R = ls.renders[r];
        const ViewConst &cv = views[R.camera_view];
        const int nct = cv.tiles_x * cv.tiles_y;
        const float *part = ls.part_render + R.part_off + (long long)slot * nct * 3;
#pragma unroll 4
        for (int q = u % cut * 256 + (int)threadIdx.x; q < nct; q += cut * 256)
#pragma unroll
            for (int k = 0; k < 3; ++k) acc[k] += part[3 * q + k];
    }
    block_sum_store<4>(acc, ls.gl_part + ((long long)l * kGlightBlocks + blk) * 3);
}

// Rows of the listed triangles.  Large ones: a workgroup per item sums its
// pairs' rows; a triangle of one item gets its row stored, the items of a
// larger one are added to its row, which the backward's setup cleared, as they
// finish (a workgroup per triangle, in order, took 126 us at 1080p).  Those
// of kOwnRows + 1 to kBigBin pairs: half a wave each, a value of the row a
// lane, the flagged rows added in order (as single lanes of the gather read
// them, 32 rows were 32 dependent rounds: tiny cube 17 -> 5 us).
__global__ __launch_bounds__(256) void large_reduce_kernel(const ViewConst *__restrict__ views, int L,
                                                           const TriSetup *__restrict__ setup, LargeLists large,
                                                           const DevCounters *counters,
                                                           const unsigned *__restrict__ pair_off, unsigned capacity,
                                                           const unsigned char *__restrict__ pair_flag,
                                                           const float *__restrict__ pair_sums,
                                                           float *__restrict__ gtri, LightSum ls) {
    if ((int)blockIdx.x >= kLargeBlocks) {
        const int q = (int)blockIdx.x - kLargeBlocks;
        light_partials(q / kGlightBlocks, q % kGlightBlocks, views, ls);
        return;
    }
    __shared__ float part[4][kNV];
    for_large_items(large, counters, (int)blockIdx.x, kLargeBlocks,
                    [&](unsigned t) { return pair_off[t + 1] - pair_off[t]; },
                    [&](unsigned t, unsigned q0, unsigned n) {
                        const unsigned a = pair_off[t];
                        if (a + n > capacity) return;                       // overflowed: filled by atomics
                        constexpr int PER = kLargeChunk / 256;
                        bool on[PER];
#pragma unroll
                        for (int k = 0; k < PER; ++k) {
                            const unsigned q = q0 + 256u * k + threadIdx.x;
                            on[k] = q < n && pair_flag[a + q];
                        }
                        float4 acc[kRow / 4];
#pragma unroll
                        for (int i = 0; i < kRow / 4; ++i) acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                        for (int k = 0; k < PER; ++k) {
                            if (!on[k]) continue;
                            const float4 *row = (const float4 *)(pair_sums + (size_t)(a + q0 + 256u * k + threadIdx.x) * kRow);
#pragma unroll
                            for (int i = 0; i < kRow / 4; ++i) {
                                const float4 r = row[i];
                                acc[i].x += r.x; acc[i].y += r.y; acc[i].z += r.z; acc[i].w += r.w;
                            }
                        }
                        float v[kNV];
#pragma unroll
                        for (int i = 0; i < kNV; ++i) {
                            const float4 c = acc[row_slot(i) / 4];
                            v[i] = row_slot(i) % 4 == 0 ? c.x : row_slot(i) % 4 == 1 ? c.y : row_slot(i) % 4 == 2 ? c.z : c.w;
                        }
                        const int lane = (int)(threadIdx.x & 63), i = lane >> 1;
                        const float s = wave_sum_multi(v);
                        __syncthreads();
                        if ((lane & 1) == 0 && i < kNV) part[threadIdx.x >> 6][i] = s;
                        __syncthreads();
                        if (threadIdx.x < kNV) {
                            const int q = (int)threadIdx.x;
                            const float total = (part[0][q] + part[1][q]) + (part[2][q] + part[3][q]);
                            float *dst = gtri + (size_t)t * kRow + row_slot(q);
                            // light views' rows have no albedo terms
                            if (q >= 18 && setup[t].pad2[0] < L) return;
                            if (n <= kLargeChunk) *dst = total;
                            else atomic_add_f32(dst, total);
                        }
                    });
    const unsigned nmedium = counters->medium_len;
    const int half = (int)(threadIdx.x & 63) >> 5, i = (int)(threadIdx.x & 31);
    for (unsigned o = blockIdx.x * 8u + (threadIdx.x >> 5); __ballot(o < nmedium) != 0ull; o += kLargeBlocks * 8u) {
        const unsigned t = o < nmedium ? large.medium[o] : 0u;
        const unsigned a = pair_off[t], n = o < nmedium ? pair_off[t + 1] - a : 0u;
        const bool live = n > 0 && a + n <= capacity;
        const unsigned long long m2 = __ballot(live && (unsigned)i < n && pair_flag[a + (live ? i : 0)]);
        unsigned m = (unsigned)(half ? m2 >> 32 : m2);
        if (!live || i >= kRow) continue;
        const float *rows = pair_sums + (size_t)a * kRow + i;
        float acc = 0.f;
        while (m) {
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = m ? rows[(size_t)(__ffs((int)m) - 1) * kRow] : 0.f;
                m &= m - 1;
            }
            acc += v[0]; acc += v[1]; acc += v[2]; acc += v[3];
        }
        gtri[(size_t)t * kRow + i] = acc;
    }
}

// Albedo gradient per face: sum over the camera views of its scene.  Run by
// the workgroups of the vertex gather's launch past its vertex blocks
// (column bx of scene b).
__device__ __forceinline__ void albedo_gather_block(const ViewConst *__restrict__ views, int L, int b, int bx,
                                                    const int *__restrict__ scene_face_off,
                                                    const int *__restrict__ scene_views_off,
                                                    const int *__restrict__ scene_views,
                                                    const unsigned *__restrict__ pair_off, unsigned capacity,
                                                    const unsigned char *__restrict__ pair_flag,
                                                    const float *__restrict__ pair_sums,
                                                    const float *__restrict__ gtri, float *__restrict__ galbedo,
                                                    int C) {
    const int fl = bx * blockDim.x + threadIdx.x;
    if (fl >= scene_face_off[b + 1] - scene_face_off[b]) return;
    float acc[3] = {0, 0, 0};
    for (int s = scene_views_off[b]; s < scene_views_off[b + 1]; ++s) {
        const int vi = scene_views[s];
        if (vi < L) continue;
        const unsigned t = (unsigned)(views[vi].setup_off + fl), p0 = pair_off[t], p1 = pair_off[t + 1];
        TriRows r = tri_rows(t, p0, p1, flag_word(pair_flag + (p1 <= capacity ? p0 : 0u)), capacity, pair_sums, gtri);
        while (r.mask) {
            const int j = __ffs((int)r.mask) - 1;
            r.mask &= r.mask - 1;
            for (int c = 0; c < C; ++c) acc[c] += r.rows[(size_t)j * kRow + row_slot(18 + c)];
        }
    }
    for (int c = 0; c < C; ++c) galbedo[(size_t)(scene_face_off[b] + fl) * C + c] = acc[c];
}

// Corners whose records a lane gathers together, and the number up to which it
// does so itself: a vertex of a closed mesh has about six, the pole of a UV
// sphere one per longitude, whose records past the first kOwnCorners are
// gathered by the whole wave.  (8 or 4 at a time: 58 and 53 us against 52 on 64
// scenes, registers against round trips.)
constexpr int kCorners = 6, kOwnCorners = 24;

// Six terms (world x y z, clip x y w) of up to kCorners triangle corners e[]
// (triangle << 2 | corner, -1: none) of one view: the first row of every
// corner in flight together, then every second one, and so on.  Corners with
// no row left read an all-zero record (zero_rec), so that no load sits behind
// a branch.  Uniform call.
template <int N>
__device__ __forceinline__ void gather_corners(const int (&e)[N], int soff, unsigned capacity,
                                               const unsigned *__restrict__ pair_off,
                                               const unsigned char *__restrict__ pair_flag,
                                               const float *__restrict__ pair_sums, const float *__restrict__ gtri,
                                               const float *__restrict__ zero_rec, float (&g)[6]) {
    unsigned p0[N], p1[N], w[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const unsigned t = (unsigned)(soff + (max(e[k], 0) >> 2));
        p0[k] = pair_off[t];
        p1[k] = pair_off[t + 1];
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        if (e[k] < 0) p0[k] = p1[k] = 0u;
        w[k] = flag_word(pair_flag + (p1[k] <= capacity ? p0[k] : 0u));
    }
    TriRows r[N];
#pragma unroll
    for (int k = 0; k < N; ++k)
        r[k] = tri_rows((unsigned)(soff + (max(e[k], 0) >> 2)), p0[k], p1[k], w[k], capacity, pair_sums, gtri);
    for (;;) {
        unsigned any = 0;
#pragma unroll
        for (int k = 0; k < N; ++k) any |= r[k].mask;
        if (__ballot(any != 0) == 0ull) break;
        float4 a[N];
        float2 b[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const float *rec = r[k].mask ? r[k].rows + (size_t)(__ffs((int)r[k].mask) - 1) * kRow + (e[k] & 3) * 8 : zero_rec;
            r[k].mask &= r[k].mask - 1;       // 0 stays 0
            a[k] = *(const float4 *)rec;
            b[k] = *(const float2 *)(rec + 4);
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            g[0] += a[k].x; g[1] += a[k].y; g[2] += a[k].z;
            g[3] += a[k].w; g[4] += b[k].x; g[5] += b[k].y;
        }
    }
}

// The gradient of light l by a wave: the vertex workgroups' shares and
// light_partials' sums in a fixed order.
__device__ __forceinline__ void finish_light(const ViewConst &v, int l, const float *part_gm, const LightSum &ls) {
    const int lane = (int)(threadIdx.x & 63), nblk = (v.nverts + 63) / 64;
    float acc[3] = {0.f, 0.f, 0.f};
    const float *part = part_gm + (long long)v.part_gm_off * 3;
    static_assert(kGlightBlocks <= 64, "a lane each");
    if (lane < kGlightBlocks)
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[k] = ls.gl_part[((long long)l * kGlightBlocks + lane) * 3 + k];
#pragma unroll 4
    for (int q = lane; q < nblk; q += 64)
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[k] += part[3 * q + k];
    const float t = wave_sum_multi(acc);
    if ((lane & 15) == 0 && lane < 48) ls.gparams[3 * l + (lane >> 4)] = t;
}

// Per vertex: sum its triangle corners' terms over every view of its scene,
// add the silhouette clip terms, map clip terms through M^T; per light view
// the wave's share of dL/dM is written to part_gm.  With LIGHTS the scene's
// last workgroup to finish (done, cleared by the backward's setup) adds those of
// each light to light_partials' sums, else light_sum_kernel does.  A workgroup takes
// 64 vertices, a vertex a lane, and its waves share the views.  Bound by the
// latency of the chain corner -> pair range -> flags -> rows.  With the rows of
// up to four pairs read here, no pass writes a row per triangle: with the
// reduction before it, 64 scenes 150 -> 76 us; 24 views of a 50k-vertex sphere
// whose poles have 316 corners 744 -> 91.
template <bool LIGHTS>
__global__ __launch_bounds__(256) void vertex_gather_kernel(
    const ViewConst *__restrict__ views, int L, const int *__restrict__ scene_vert_off,
    const int *__restrict__ scene_views_off, const int *__restrict__ scene_views, const int *__restrict__ vc_off,
    const int *__restrict__ vc_list, const float *__restrict__ verts, const unsigned *__restrict__ pair_off,
    unsigned capacity, const unsigned char *__restrict__ pair_flag, const float *__restrict__ pair_sums,
    const float *__restrict__ gtri, const float *__restrict__ zero_rec, const float4 *__restrict__ gclip,
    float *__restrict__ gverts, float *part_gm, const float *__restrict__ jac, int vx,
    const int *__restrict__ scene_face_off, float *__restrict__ galbedo, int C, LightSum ls) {
    const int b = blockIdx.y;
    if ((int)blockIdx.x >= vx) {                               // the albedo gather's workgroups
        albedo_gather_block(views, L, b, (int)blockIdx.x - vx, scene_face_off, scene_views_off, scene_views, pair_off,
                            capacity, pair_flag, pair_sums, gtri, galbedo, C);
        return;
    }
    const int nv = scene_vert_off[b + 1] - scene_vert_off[b];
    const int nblk = max((nv + 63) / 64, 1);                 // a scene without vertices still finishes its lights
    if ((int)blockIdx.x >= nblk) return;                     // whole workgroup
    __shared__ float sum[3][3][64];
    const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6), nwaves = (int)(blockDim.x >> 6);
    const int vl = blockIdx.x * 64 + lane;
    const bool in = vl < nv;
    const int gv_idx = scene_vert_off[b] + (in ? vl : 0);
    float x[3] = {0, 0, 0};
    if (in)
        for (int k = 0; k < 3; ++k) x[k] = verts[3 * (size_t)gv_idx + k];
    float gv[3] = {0, 0, 0};
    const int c0 = in ? vc_off[gv_idx] : 0, c1 = in ? vc_off[gv_idx + 1] : 0;
    int held[kCorners];                        // loaded once for every view
#pragma unroll
    for (int k = 0; k < kCorners; ++k) held[k] = c0 + k < c1 ? vc_list[c0 + k] : -1;
    const int own = min(c1, c0 + kOwnCorners);
    const unsigned long long many = __ballot(c1 > own);
    const int views_end = scene_views_off[b + (nv > 0 ? 1 : 0)];
    for (int s = scene_views_off[b] + wave; s < views_end; s += nwaves) {
        const int vi = scene_views[s];
        const ViewConst &v = views[vi];
        const int soff = v.setup_off;
        const float4 ga = gclip[v.clip_off + (in ? vl : 0)];     // silhouette terms, issued early
        float g[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        gather_corners(held, soff, capacity, pair_off, pair_flag, pair_sums, gtri, zero_rec, g);
        for (int c = c0 + kCorners; __ballot(c < own) != 0ull; c += kCorners) {
            int e[kCorners];
#pragma unroll
            for (int k = 0; k < kCorners; ++k) e[k] = c + k < own ? vc_list[c + k] : -1;
            gather_corners(e, soff, capacity, pair_off, pair_flag, pair_sums, gtri, zero_rec, g);
        }
        for (unsigned long long m = many; m; m &= m - 1) {
            const int l = __ffsll(m) - 1;
            const int q0 = __builtin_amdgcn_readlane(own, l), q1 = __builtin_amdgcn_readlane(c1, l);
            float h[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            for (int q = q0; q < q1; q += 128) {
                const int e[2] = {q + lane < q1 ? vc_list[q + lane] : -1, q + 64 + lane < q1 ? vc_list[q + 64 + lane] : -1};
                gather_corners(e, soff, capacity, pair_off, pair_flag, pair_sums, gtri, zero_rec, h);
            }
            const float t = wave_sum_multi(h);           // lane 8k: total of term k
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const float tk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), k << kSumShift<6>));
                if (lane == l) g[k] += tk;
            }
        }
        float gc[3] = {g[3], g[4], g[5]};
        if (in) {
            gc[0] += ga.x; gc[1] += ga.y; gc[2] += ga.w;
        }
        const float *M = v.M;
#pragma unroll
        for (int k = 0; k < 3; ++k) gv[k] += g[k] + ((M[k] * gc[0] + M[4 + k] * gc[1]) + M[12 + k] * gc[2]);
        if (vi < L) {
            // dL/dM = (gc_x, gc_y, 0, gc_w) outer [x, 1], pulled back to the light parameter
            const float xh[4] = {x[0], x[1], x[2], in ? 1.f : 0.f};
            const float *J = jac + (size_t)kJac * vi;
            float gp[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                float a = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    a += xh[k] * ((gc[0] * J[3 * k + j] + gc[1] * J[3 * (4 + k) + j]) + gc[2] * J[3 * (12 + k) + j]);
                gp[j] = a;
            }
            const float t = wave_sum_multi(gp);
            if ((lane & 15) == 0 && lane < 48) part_gm[((long long)v.part_gm_off + blockIdx.x) * 3 + (lane >> 4)] = t;
        }
    }
    if (wave > 0)
#pragma unroll
        for (int k = 0; k < 3; ++k) sum[wave - 1][k][lane] = gv[k];
    __shared__ unsigned before;
    if (LIGHTS || nwaves > 1) __syncthreads();
    // releases the workgroup's shares (stored before the barrier) and, in the last
    // one, acquires the others'
    if constexpr (LIGHTS)
        if (threadIdx.x == 0)
            before = __hip_atomic_fetch_add(ls.done + b, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (wave == 0) {
        for (int w = 1; w < nwaves; ++w)
#pragma unroll
            for (int k = 0; k < 3; ++k) gv[k] += sum[w - 1][k][lane];
        if (in)
            for (int k = 0; k < 3; ++k) gverts[3 * (size_t)gv_idx + k] = gv[k];
    }
    if constexpr (LIGHTS) {
        __syncthreads();
        if (before != (unsigned)nblk - 1u) return;
        for (int s = scene_views_off[b] + wave; s < scene_views_off[b + 1]; s += nwaves) {
            const int vi = scene_views[s];
            if (vi < L) finish_light(views[vi], vi, part_gm, ls);
        }
    }
}

// The lights' gradients where the gather does not finish them, a wave each.
__global__ __launch_bounds__(64) void light_sum_kernel(const ViewConst *__restrict__ views, const float *part_gm,
                                                       LightSum ls) {
    finish_light(views[blockIdx.x], (int)blockIdx.x, part_gm, ls);
}

// ----------------------------------------------------------------------------- pose

__host__ __device__ inline Dual3 dsin(const Dual3 &a) {
    const double s = sin(a.v), c = cos(a.v);
    return Dual3{s, {c * a.d[0], c * a.d[1], c * a.d[2]}};
}
__host__ __device__ inline Dual3 dcos(const Dual3 &a) {
    const double s = sin(a.v), c = cos(a.v);
    return Dual3{c, {-s * a.d[0], -s * a.d[1], -s * a.d[2]}};
}
__host__ __device__ inline double dsin(double a) { return sin(a); }
__host__ __device__ inline double dcos(double a) { return cos(a); }

// Rotation matrix of an axis-angle vector (Rodrigues): I + sin(t)/t K + (1-cos t)/t^2 K^2.
template <class T>
__device__ inline void rodrigues(const T r[3], T Rm[9]) {
    const T th2 = (r[0] * r[0] + r[1] * r[1]) + r[2] * r[2];
    const T zero = mkT<T>(0.0);
    const T K[9] = {zero, -r[2], r[1], r[2], zero, -r[0], -r[1], r[0], zero};
    T K2[9];
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) {
            T s = zero;
            for (int k = 0; k < 3; ++k) s = s + K[3 * a + k] * K[3 * k + c];
            K2[3 * a + c] = s;
        }
    const bool small = val(th2) < 1e-24;
    for (int k = 0; k < 9; ++k) Rm[k] = K[k];
    if (!small) {
        const T th = dsqrt(th2);
        const T A = dsin(th) / th;
        const T Bc = (mkT<T>(1.0) - dcos(th)) / th2;
        for (int k = 0; k < 9; ++k) Rm[k] = A * K[k] + Bc * K2[k];
    }
    Rm[0] = Rm[0] + mkT<T>(1.0);
    Rm[4] = Rm[4] + mkT<T>(1.0);
    Rm[8] = Rm[8] + mkT<T>(1.0);
}

__global__ void pose_kernel(const int *__restrict__ vert_off, const int *__restrict__ pose_counts,
                            const float *__restrict__ centers, const float *__restrict__ local,
                            const float *__restrict__ poses, float *__restrict__ world) {
    const int b = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int nv = vert_off[b + 1] - vert_off[b];
    if (i >= nv) return;
    const size_t gi = (size_t)(vert_off[b] + i);
    const float *src = local + 3 * gi;
    float *dst = world + 3 * gi;
    if (i >= pose_counts[b]) {
        dst[0] = src[0]; dst[1] = src[1]; dst[2] = src[2];
        return;
    }
    const double r[3] = {poses[6 * b], poses[6 * b + 1], poses[6 * b + 2]};
    double Rm[9];
    rodrigues<double>(r, Rm);
    for (int a = 0; a < 3; ++a) {
        const double acc = ((Rm[3 * a] * src[0] + Rm[3 * a + 1] * src[1]) + Rm[3 * a + 2] * src[2]) +
                           (double)centers[3 * b + a] + (double)poses[6 * b + 3 + a];
        dst[a] = (float)acc;
    }
}

__global__ __launch_bounds__(256) void pose_backward_kernel(const int *__restrict__ vert_off,
                                                            const int *__restrict__ pose_counts,
                                                            const float *__restrict__ local,
                                                            const float *__restrict__ poses,
                                                            const float *__restrict__ gworld,
                                                            float *__restrict__ gposes) {
    const int b = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x * blockDim.x >= (unsigned)pose_counts[b]) return;     // whole workgroup idle
    const bool in = i < pose_counts[b];
    Dual3 r[3];
    for (int k = 0; k < 3; ++k) {
        r[k].v = poses[6 * b + k];
        for (int q = 0; q < 3; ++q) r[k].d[q] = k == q ? 1.0 : 0.0;
    }
    Dual3 Rm[9];
    rodrigues<Dual3>(r, Rm);
    float out[6] = {0, 0, 0, 0, 0, 0};
    if (in) {
        const size_t gi = (size_t)(vert_off[b] + i);
        const float *v = local + 3 * gi;
        const float *g = gworld + 3 * gi;
        for (int q = 0; q < 3; ++q) {
            double acc = 0;
            for (int a = 0; a < 3; ++a)
                acc += g[a] * ((Rm[3 * a].d[q] * v[0] + Rm[3 * a + 1].d[q] * v[1]) + Rm[3 * a + 2].d[q] * v[2]);
            out[q] = (float)acc;
        }
        out[3] = g[0]; out[4] = g[1]; out[5] = g[2];
    }
    __shared__ float part[4][6];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int k = 0; k < 6; ++k) {
        const float s = wave_sum(out[k]);
        if (lane == 0) part[wid][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const float s = (part[0][threadIdx.x] + part[1][threadIdx.x]) + (part[2][threadIdx.x] + part[3][threadIdx.x]);
        atomic_add_f32(gposes + 6 * b + threadIdx.x, s);
    }
}

// ----------------------------------------------------------------------------- launchers

hipError_t launch_aa_camera_backward(const ViewConst *views, int L, int Cm, int max_regions, int max_renders,
                                     const RenderConst *renders, const int *cam_renders_off, const int *cam_renders,
                                     const TriSetup *setup, const int *faces, const unsigned char *silm, const float *verts,
                                     const unsigned long long *keys, const unsigned char *aa_flag, const float *img0,
                                     const float *gimg, float *gimg0, float4 *gclip, int C, hipStream_t s) {
    if (Cm == 0 || max_renders == 0) return hipSuccess;
    const int chunk = render_chunk(max_renders, (long long)max_regions * Cm);
    const dim3 grid(max_regions, Cm, (max_renders + chunk - 1) / chunk);
#define DSM_AACB(CC)                                                                                                 \
    hipLaunchKernelGGL(aa_camera_backward_kernel<CC>, grid, dim3(64), 0, s, views, L, renders, cam_renders_off,     \
                       cam_renders, chunk, setup, faces, silm, verts, keys, aa_flag, img0, gimg, gimg0, gclip)
    if (C == 1) DSM_AACB(1);
    else DSM_AACB(3);
#undef DSM_AACB
    return hipGetLastError();
}

hipError_t launch_lookup_backward(int tile, const ViewConst *views, int L, int Cm, int max_tiles,
                                  const RenderConst *renders, const int *cam_renders_off, const int *cam_renders,
                                  const int *render_lights, const TriVerts *tv, const unsigned long long *keys,
                                  const float *maps, const float *gimg0, float *gmaps, const TriSetup *setup,
                                  const unsigned *tile_start, const unsigned *bins, const unsigned *bin_pair,
                                  unsigned char *pair_flag, float *pair_sums, float *gtri, float *part_render, int C,
                                  const float *jac, const unsigned *pair_off, unsigned capacity, hipStream_t s) {
    if (Cm == 0 || max_tiles == 0) return hipSuccess;
    const dim3 grid(max_tiles, Cm);
#define DSM_LB(TT, CC)                                                                                             \
    hipLaunchKernelGGL((lookup_backward_kernel<TT, CC>), grid, dim3(TileShape<TT>::NT), 0, s, views, L, renders,  \
                       cam_renders_off, cam_renders, render_lights, tv, keys, maps, gimg0, gmaps, setup,          \
                       tile_start, bins, bin_pair, pair_flag, pair_sums, gtri, part_render, jac, pair_off, capacity)
#define DSM_LB_C(TT)          \
    if (C == 1) DSM_LB(TT, 1); \
    else DSM_LB(TT, 3)
    if (tile == 8) { DSM_LB_C(8); }
    else if (tile == 16) { DSM_LB_C(16); }
    else { DSM_LB_C(32); }
#undef DSM_LB_C
#undef DSM_LB
    return hipGetLastError();
}

hipError_t launch_light_backward(int tile, const ViewConst *views, int L, int max_tiles, const TriSetup *setup,
                                 const int *faces, const unsigned char *silm, const float *verts, const TriVerts *tv,
                                 const unsigned long long *keys, const unsigned char *aa_flag, const float *F0, const float *gF1,
                                 float4 *gclip,
                                 const unsigned *tile_start, const unsigned *bins, const unsigned *bin_pair,
                                 unsigned char *pair_flag, float *pair_sums, float *gtri, float *part_light,
                                 const float *jac, const unsigned *pair_off, unsigned capacity, hipStream_t s) {
    if (L == 0 || max_tiles == 0) return hipSuccess;
    const dim3 grid(max_tiles, L);
#define DSM_LIB(TT)                                                                                                  \
    hipLaunchKernelGGL((light_backward_kernel<TT>), grid, dim3(TileShape<TT>::NT), 0, s, views, setup, faces, silm,  \
                       verts, tv, keys, aa_flag, F0, gF1, gclip, tile_start, bins, bin_pair, pair_flag, pair_sums, \
                       gtri, part_light, jac, pair_off, capacity)
    if (tile == 8) DSM_LIB(8);
    else if (tile == 16) DSM_LIB(16);
    else DSM_LIB(32);
#undef DSM_LIB
    return hipGetLastError();
}

hipError_t launch_vertex_gradients(const ViewConst *views, int L, int B, int max_verts, int max_faces, int max_views,
                                   int ntri, unsigned capacity, const TriSetup *setup, const LargeLists &large,
                                   const DevCounters *counters, const int *scene_vert_off, const int *scene_face_off,
                                   const int *scene_views_off, const int *scene_views, const int *vc_off,
                                   const int *vc_list, const unsigned *pair_off, const unsigned char *pair_flag,
                                   const float *pair_sums, float *gtri, const float *zero_rec, const float *verts,
                                   const float4 *gclip, float *gverts, float *part_gm, float *galbedo, int C,
                                   const float *jac, const LightSum &ls, hipStream_t s) {
    if (ntri > 0 || L > 0)
        hipLaunchKernelGGL(large_reduce_kernel, dim3(kLargeBlocks + kGlightBlocks * L), dim3(256), 0, s, views, L, setup,
                           large, counters, pair_off, capacity, pair_flag, pair_sums, gtri, ls);
    // one launch: the vertex gather's workgroups, then the albedo gather's;
    // a wave per view of the scene, up to four
    const int nt = 64 * std::min(std::max(max_views, 1), 4);
    const int vx = std::max((max_verts + 63) / 64, 1), fx = (galbedo && max_faces > 0) ? (max_faces + nt - 1) / nt : 0;
    if (B == 0) return hipGetLastError();
#define DSM_GATHER(LIGHTS)                                                                                          \
    hipLaunchKernelGGL(vertex_gather_kernel<LIGHTS>, dim3(vx + fx, B), dim3(nt), 0, s, views, L, scene_vert_off,   \
                       scene_views_off, scene_views, vc_off, vc_list, verts, pair_off, capacity, pair_flag,        \
                       pair_sums, gtri, zero_rec, gclip, gverts, part_gm, jac, vx, scene_face_off, galbedo, C, ls)
    // On few workgroups finishing the lights in the gather saves a launch: tiny cube
    // 118.3 -> 116.4 us, icosphere 156.7 -> 155.8.  With more, the release of each
    // (a write-back of its XCD's L2) keeps the workgroup's place: four lights and
    // views, 111 workgroups 233.0 us a pass against 231.6 with the launch; one of
    // each, 160: 144.7 against 143.1, 240: 146.4 against 144.2.
    constexpr long long kFinishBlocks = 64;
    if (L > 0 && (long long)vx * B <= kFinishBlocks) DSM_GATHER(true);
    else {
        DSM_GATHER(false);
        if (L > 0) hipLaunchKernelGGL(light_sum_kernel, dim3(L), dim3(64), 0, s, views, part_gm, ls);
    }
#undef DSM_GATHER
    return hipGetLastError();
}

hipError_t launch_pose(const int *scene_vert_off, const int *pose_counts, const float *pose_centers, int B,
                       int max_verts, const float *local, const float *poses, float *world, hipStream_t s) {
    hipLaunchKernelGGL(pose_kernel, dim3((max_verts + 255) / 256, B), dim3(256), 0, s, scene_vert_off, pose_counts,
                       pose_centers, local, poses, world);
    return hipGetLastError();
}

hipError_t launch_pose_backward(const int *scene_vert_off, const int *pose_counts, int B, int max_verts,
                                const float *local, const float *poses, const float *gworld, float *gposes,
                                hipStream_t s) {
    hipLaunchKernelGGL(pose_backward_kernel, dim3((max_verts + 255) / 256, B), dim3(256), 0, s, scene_vert_off,
                       pose_counts, local, poses, gworld, gposes);
    return hipGetLastError();
}

}  // namespace dsm
