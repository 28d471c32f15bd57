// Rasterization of every view of a batch (light views into shadow maps, Eq. 1;
// camera views for deferred shading): vertex transform, fixed-point triangle
// setup, tile binning, and a tile rasterizer producing a 64-bit
// depth|triangle-id visibility buffer (the nearest surface per sample, ties
// to the lower triangle index).
//
// Coverage conventions (shared with no other code; stated here in full):
//  * clip = M [x,1] per row as ((m0*x + m1*y) + m2*z) + m3 in float32 (the
//    library is built without contraction, so no fused multiply-add);
//  * sx = (x/w + 1) * (W/2), sy = (1 - y/w) * (H/2); X = rint(256 sx),
//    Y = rint(256 sy); pixel (i,j) is sampled at (256 i + 128, 256 j + 128);
//  * a triangle is culled when a vertex has w <= 0, z/w < -1, or a screen
//    coordinate outside (-32768, 32768); it is re-oriented to positive doubled
//    area A (2nd and 3rd vertex swapped when A < 0), A == 0 is skipped;
//  * edge e is opposite vertex e, E_e = dx (py - ya) - dy (px - xa) for the
//    directed edge a -> b; a sample on an edge belongs to the triangle only
//    for top (dy == 0, dx > 0) or left (dy < 0) edges;
//  * z01 = 0.5 z/w + 0.5 per vertex, interpolated (z0 + b1 (z1-z0)) + b2 (z2-z0)
//    with b_e = f32(E_e) rA, rA the correctly rounded float32 1 / A; samples with
//    z01 outside [0,1] are dropped;
//  * key = bits(z01) << 32 | local triangle index, minimum wins.
#include "dsm_internal.h"
#include "frames.h"

namespace dsm {

// ----------------------------------------------------------------------------- light frames

// The Jacobian of (M[16], pos[3], dir[3]) with respect to the three
// parameter components (forward-mode dual numbers), [22][3] per light: the
// reverse pass pulls every light-frame gradient back to the parameter as
// soon as it is formed.
__device__ void light_jacobian(const CamStatic &cam, const float *param, float *J) {
    Dual3 pd[3];
    for (int i = 0; i < 3; ++i) {
        pd[i].v = param[i];
        for (int j = 0; j < 3; ++j) pd[i].d[j] = (i == j) ? 1.0 : 0.0;
    }
    Dual3 Md[16], posd[3], dird[3];
    light_frame<Dual3>(cam, pd, Md, posd, dird);
    for (int j = 0; j < 3; ++j) {
        for (int i = 0; i < 16; ++i) J[3 * i + j] = (float)Md[i].d[j];
        for (int i = 0; i < 3; ++i) {
            J[3 * (16 + i) + j] = (float)posd[i].d[j];
            J[3 * (19 + i) + j] = (float)dird[i].d[j];
        }
    }
}

// One thread per light: the light camera from its float32 parameter, in
// float64, rounded to float32 for the rest of the pipeline; with jac, also
// the frame's Jacobian.  Workgroups from nf on clear the words z1[0, n1) and
// z2[0, n2) instead, and those rows (the pass's counters and accumulators: one
// launch for all of it).
__global__ void light_frames_kernel(ViewConst *views, const CamStatic *cams, const float *params, int L,
                                    float *zc_out, float *jac, int nf, unsigned *z1, size_t n1, unsigned *z2,
                                    size_t n2, ClearRows rows) {
    if ((int)blockIdx.x >= nf) {
        const size_t stride = (size_t)(gridDim.x - nf) * blockDim.x;
        const size_t first = (size_t)(blockIdx.x - nf) * blockDim.x + threadIdx.x;
        for (size_t i = first; i < n1 + n2; i += stride) {
            if (i < n1) z1[i] = 0u;
            else z2[i - n1] = 0u;
        }
        if (rows.rows) {
            if (rows.pairs && *rows.pairs == kPairEnd) {
                for (size_t i = first; i < 24 * (size_t)rows.ntri; i += stride) rows.rows[i] = 0.f;
                return;
            }
            const size_t la = *rows.len_a, lb = *rows.len_b;
            for (size_t i = first; i < 24 * (la + lb); i += stride) {
                const size_t o = i / 24;
                rows.rows[(size_t)(o < la ? rows.list_a[o] : rows.list_b[o - la]) * 24 + i % 24] = 0.f;
            }
        }
        return;
    }
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= L) return;
    const double p[3] = {params[3 * l], params[3 * l + 1], params[3 * l + 2]};
    double M[16], pos[3], dir[3];
    light_frame<double>(cams[l], p, M, pos, dir);
    ViewConst &v = views[l];
    for (int i = 0; i < 16; ++i) v.M[i] = (float)M[i];
    for (int i = 0; i < 3; ++i) {
        v.pos[i] = (float)pos[i];
        v.dir[i] = (float)dir[i];
    }
    v.zc = (float)light_reference_depth(cams[l], p);
    if (zc_out) zc_out[l] = v.zc;
    if (jac) light_jacobian(cams[l], params + 3 * l, jac + (size_t)kJac * l);
}

// ----------------------------------------------------------------------------- setup

__device__ __forceinline__ int floor_div256(int a) { return a >= 0 ? (a >> 8) : -((-a + 255) >> 8); }

// Workgroups of the triangle passes (setup, bin count, bin fill) take runs of
// kTriRun triangles of one view (TriBlock, in the order of the per-(view,
// triangle) arrays), a triangle a thread.
constexpr int kTriThreads = kTriRun;

// Exclusive scan over the workgroup's PPT * 256 values, value k of thread tid
// at position k * 256 + tid; *total: their sum.  SAT: every sum stays at the
// largest value once it passes it.  Uniform call.
template <int PPT, bool SAT = false>
__device__ __forceinline__ void tri_block_scan(const unsigned (&v)[PPT], unsigned (&out)[PPT], unsigned *total) {
    constexpr int NW = kTriThreads / 64;
    __shared__ unsigned sum[PPT][NW];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        unsigned x = v[k];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned y = __shfl_up(x, o, 64);
            if (lane >= o) x = SAT ? add_sat(x, y) : x + y;
        }
        if (lane == 63) sum[k][wid] = x;
        if (SAT) {
            const unsigned before = __shfl_up(x, 1, 64);
            out[k] = lane > 0 ? before : 0u;
        } else {
            out[k] = x - v[k];
        }
    }
    __syncthreads();
    unsigned all = 0;
#pragma unroll
    for (int k = 0; k < PPT; ++k)
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (w == wid) out[k] = SAT ? add_sat(out[k], all) : out[k] + all;
            all = SAT ? add_sat(all, sum[k][w]) : all + sum[k][w];
        }
    *total = all;
}

// Tiles of the pixel box [x0, x1] x [y0, y1] (empty: x1 < x0).
struct TileBox {
    int tx0, ty0, ntx;
    unsigned n;
};
__device__ __forceinline__ TileBox tile_box(int x0, int x1, int y0, int y1, int shift) {
    TileBox b;
    b.tx0 = x0 >> shift;
    b.ty0 = y0 >> shift;
    b.ntx = (x1 >> shift) - b.tx0 + 1;
    b.n = x0 <= x1 && y0 <= y1 ? (unsigned)(b.ntx * ((y1 >> shift) - b.ty0 + 1)) : 0u;
    return b;
}
__device__ __forceinline__ TileBox tile_box(const TriSetup &s, int shift) {
    return tile_box(s.bx0, s.bx1, s.by0, s.by1, shift);
}

// Triangles with at most kBigBin tiles are binned by their wave.  The setup
// lists the larger ones (large_list) and cuts them into items of kLargeChunk
// pairs, a workgroup's work each, so that a ground polygon's 65,536 tiles are
// 64 workgroups' work and not one's.  The items fit unless the pairs exceed
// the bin capacity; then the passes walk large_list instead (for_large_items).
__device__ __forceinline__ void list_large(unsigned t, unsigned n, const LargeLists &l, DevCounters *counters) {
    l.list[atomicAdd(&counters->large_len, 1u)] = t;
    const unsigned k = (n + kLargeChunk - 1) / kLargeChunk;
    const unsigned long long at = atomicAdd(&counters->item_len, (unsigned long long)k);
    for (unsigned q = 0; q < k && at + q < l.item_cap; ++q) l.items[at + q] = make_uint2(t, q * kLargeChunk);
}

// Per (view, triangle): the corners' clip coordinates (in the fixed order of
// clip_of), the fixed-point record, the facing byte and the number of tiles,
// scanned within the workgroup (pair_local, block totals).  The first view of
// each scene also writes the faces' TriVerts records: world positions and
// albedo gathered once, so that per-pixel passes fetch one record.  Bound by
// the latency of the index -> vertex loads.
__global__ __launch_bounds__(kTriThreads) void setup_kernel(
    const ViewConst *__restrict__ views, const TriBlock *__restrict__ blocks, const int *__restrict__ faces,
    const float *__restrict__ verts, const float *__restrict__ albedo, int C, TriVerts *__restrict__ tv,
    TriSetup *__restrict__ setup, signed char *__restrict__ facing8, unsigned *__restrict__ pair_local,
    unsigned *__restrict__ block_total, unsigned long long *__restrict__ group_total, LargeLists large, int shift,
    DevCounters *counters) {
    const TriBlock blk = blocks[blockIdx.x];
    const ViewConst &v = views[blk.view];
    const float hw = 0.5f * (float)v.W, hh = 0.5f * (float)v.H;
    const int t = blk.first + (int)threadIdx.x;
    unsigned npairs[1] = {0u}, nculled = 0, nbad = 0;
    if (t < v.nfaces) {
        const int *f = faces + 3 * (size_t)(v.face_off + t);
        int idx[3] = {f[0], f[1], f[2]};
        bool bad = false;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (idx[k] < 0 || idx[k] >= v.nverts) { bad = true; idx[k] = 0; }
        float p[3][3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) p[k][c] = verts[3 * (size_t)(v.vert_off + idx[k]) + c];
        if (v.write_tv) {
            TriVerts r;
            const float *rho = albedo + (size_t)(v.face_off + t) * C;
            r.a = make_float4(p[0][0], p[0][1], p[0][2], p[1][0]);
            r.b = make_float4(p[1][1], p[1][2], p[2][0], p[2][1]);
            r.c = make_float4(p[2][2], rho[0], C > 1 ? rho[1] : 0.f, C > 2 ? rho[2] : 0.f);
            tv[v.face_off + t] = r;
        }
        int X[3], Y[3];
        float z[3];
        bool ok = !bad;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float4 c = clip_of(v.M, p[k][0], p[k][1], p[k][2]);
            const float nx = c.x / c.w, ny = c.y / c.w, nz = c.z / c.w;
            const float sx = (nx + 1.0f) * hw;
            const float sy = (1.0f - ny) * hh;
            const bool okv = (c.w > 0.0f) && (nz >= -1.0f) && (fabsf(sx) < kGuard) && (fabsf(sy) < kGuard);
            ok = ok && okv;
            X[k] = okv ? (int)rintf(sx * 256.0f) : 0;
            Y[k] = okv ? (int)rintf(sy * 256.0f) : 0;
            z[k] = 0.5f * nz + 0.5f;
        }
        long long A = (long long)(X[1] - X[0]) * (Y[2] - Y[0]) - (long long)(Y[1] - Y[0]) * (X[2] - X[0]);
        const bool swapped = A < 0;
        if (swapped) {
            int ti = X[1]; X[1] = X[2]; X[2] = ti;
            ti = Y[1]; Y[1] = Y[2]; Y[2] = ti;
            float tz = z[1]; z[1] = z[2]; z[2] = tz;
            A = -A;
        }
        const bool valid = ok && A > 0;
        TriSetup s;
        s.A = A;
#pragma unroll
        for (int k = 0; k < 3; ++k) { s.X[k] = X[k]; s.Y[k] = Y[k]; s.z[k] = z[k]; }
        s.facing = valid ? (swapped ? -1 : 1) : 0;
        s.swapped = swapped ? 1 : 0;
        s.pad1[0] = s.pad1[1] = 0;
        s.pad2[0] = blk.view;
        s.pad2[1] = 0;
        int i0 = 1, i1 = 0, j0 = 1, j1 = 0;
        if (valid) {
            const int mnx = min(X[0], min(X[1], X[2])), mxx = max(X[0], max(X[1], X[2]));
            const int mny = min(Y[0], min(Y[1], Y[2])), mxy = max(Y[0], max(Y[1], Y[2]));
            // pixel centres 256 i + 128 inside [mnx, mxx]
            i0 = max(floor_div256(mnx - 128 + 255), 0);
            i1 = min(floor_div256(mxx - 128), v.W - 1);
            j0 = max(floor_div256(mny - 128 + 255), 0);
            j1 = min(floor_div256(mxy - 128), v.H - 1);
        }
        if (!(i0 <= i1 && j0 <= j1)) { i0 = 1; i1 = 0; j0 = 1; j1 = 0; }
        s.bx0 = (unsigned short)i0;
        s.bx1 = (unsigned short)i1;
        s.by0 = (unsigned short)j0;
        s.by1 = (unsigned short)j1;
        setup[v.setup_off + t] = s;
        facing8[v.setup_off + t] = s.facing;
        npairs[0] = tile_box(i0, i1, j0, j1, shift).n;
        if (npairs[0] > kBigBin) list_large((unsigned)(v.setup_off + t), npairs[0], large, counters);
        else if (npairs[0] > kOwnRows) large.medium[atomicAdd(&counters->medium_len, 1u)] = (unsigned)(v.setup_off + t);
        nculled += !ok && !bad ? 1u : 0u;
        nbad += bad ? 1u : 0u;
    }
    unsigned off[1], total;
    tri_block_scan(npairs, off, &total);
    if (t < v.nfaces) pair_local[v.setup_off + t] = off[0];
    if (threadIdx.x == 0) {
        block_total[blockIdx.x] = total;
        if (total) atomicAdd(&group_total[blockIdx.x / kTriGroup * kGroupStride], (unsigned long long)total);
    }
    if (__ballot(nculled + nbad != 0)) {
        if (nculled) atomicAdd(&counters->culled, (unsigned long long)nculled);
        if (nbad) atomicAdd(&counters->bad_indices, (unsigned long long)nbad);
    }
}

// ----------------------------------------------------------------------------- binning

// Pairs of triangle i are the tiles of its bounding box in row-major order,
// numbered pair_off[i] .. pair_off[i+1]-1.  The count pass counts pairs per
// tile and records each pair's slot in its tile (pair_slot, by pair); the
// fill pass scatters the triangle (and, where the backward walks bins, the
// pair) to tile start + slot, with no atomics.  Triangles whose pair range
// does not fit the bin capacity go to the overflow path instead (decided per
// triangle, so never split).

// Tile starts are scanned in blocks of kScanBlock tiles whose bases come from
// a running total, so every block keeps its own end: the start of tile t is
// at t + (t >> kScanShift), its end one further.
__device__ __forceinline__ int tile_start_at(int t) { return t + (t >> kScanShift); }

// One counter atomic per distinct g in the wave (neighbouring triangles of a
// mesh mostly share tiles): size lanes hold the leader's g, which adds size to
// the counter; a lane's slot is the old count plus its rank.  A round per
// distinct g is a serial chain, so after kSlotRounds the remaining lanes add
// their own 1, as all do where few triangles (share = false) hold the step's
// pairs: their tiles are distinct.  Uniform call (all 64 lanes).
constexpr int kSlotRounds = 24;
struct WaveSlot {
    int leader;
    unsigned rank, size;     // size: leaders only, else 0
};
__device__ __forceinline__ WaveSlot wave_slot(bool has, int g, bool share) {
    const int lane = (int)(threadIdx.x & 63);
    unsigned long long pending = share ? __ballot(has) : 0ull;
    WaveSlot s{lane, 0u, has ? 1u : 0u};
    for (int k = 0; pending && k < kSlotRounds; ++k) {
        const int leader = __ffsll(pending) - 1;
        const int gg = __builtin_amdgcn_readlane(g, leader);
        const bool mine = has && g == gg;
        const unsigned long long m = __ballot(mine);
        pending &= ~m;
        if (mine) {
            s.leader = leader;
            s.rank = (unsigned)__popcll(m & ((1ull << lane) - 1ull));
            s.size = lane == leader ? (unsigned)__popcll(m) : 0u;
        }
    }
    return s;
}

// The pairs of a wave's 64 triangles (cnt each, at most kBigBin), flattened:
// kPairSteps * 64 pairs a round in pair order, a pair a lane and step, so that
// a round's loads and atomics are in flight together.  A step's owners come
// from one bit mask of the triangles that start in it.  f(n, box, q, has) is
// called once a round by all lanes: n steps with the triangle's box, the pair
// within the triangle, whether the lane has a pair, and how many triangles
// start in the step.
struct BinItem {
    int tile0, ntx;          // first tile of the box in the global tile list, box width
    unsigned first, a, tri;  // first flat pair, first pair, setup index
};
constexpr int kPairSteps = 4;
struct BinWave {
    BinItem item[64];
    unsigned long long mask[kPairSteps];
};

template <class F>
__device__ __forceinline__ void for_wave_pairs(BinWave &w, unsigned cnt, BinItem it, F f) {
    const int lane = (int)(threadIdx.x & 63);
    unsigned x = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    const unsigned total = (unsigned)__builtin_amdgcn_readlane((int)x, 63);
    it.first = x - cnt;
    const unsigned long long some = __ballot(cnt > 0);
    const int place = __popcll(some & ((1ull << lane) - 1ull));
    if (cnt > 0) w.item[place] = it;
    int before = 0;                                   // triangles that started in earlier steps
    for (unsigned c = 0; c < total; c += 64 * kPairSteps) {
        wave_sync();
        if (lane < kPairSteps) w.mask[lane] = 0ull;
        wave_sync();
        const unsigned at = it.first - c;
        if (cnt > 0 && it.first >= c && at < 64 * kPairSteps) atomicOr(&w.mask[at >> 6], 1ull << (at & 63));
        wave_sync();
        BinItem b[kPairSteps];
        unsigned q[kPairSteps];
        bool has[kPairSteps];
        int starts[kPairSteps];
        const int n = (int)min((total - c + 63) / 64, (unsigned)kPairSteps);
#pragma unroll
        for (int u = 0; u < kPairSteps; ++u) {
            const unsigned p = c + 64 * u + (unsigned)lane;
            has[u] = p < total;
            starts[u] = 0;
            if (u < n) {                              // uniform
                const unsigned long long m = w.mask[u];
                b[u] = w.item[has[u] ? before + __popcll(m & (~0ull >> (63 - lane))) - 1 : 0];
                q[u] = p - b[u].first;
                starts[u] = __popcll(m);
                before += starts[u];
            }
        }
        f(n, b, q, has, starts);
    }
    wave_sync();
}

// q / n for q < 2^12, 1 <= n: the product with the hardware reciprocal is off
// by under 2^-10, the quotient's distance from a whole number at least 1 / 2n.
__device__ __forceinline__ unsigned small_div(unsigned q, int n) {
    return (unsigned)(((float)q + 0.5f) * __builtin_amdgcn_rcpf((float)n));
}

// Pairs [q0, q1), at most kLargeChunk, of one large triangle by the whole
// workgroup, every pair's load or atomic in flight together.
template <bool FILL>
__device__ __forceinline__ void bin_range(const ViewConst &v, const TriSetup &s, unsigned tri, unsigned a, unsigned q0,
                                          unsigned q1, int shift, unsigned *__restrict__ tile_count,
                                          unsigned *__restrict__ pair_slot, const unsigned *__restrict__ tile_start,
                                          unsigned *__restrict__ bins, unsigned *__restrict__ bin_pair) {
    constexpr int PER = kLargeChunk / kTriThreads;
    const TileBox b = tile_box(s, shift);
    int gt[PER];
    unsigned slot[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const unsigned q = q0 + (unsigned)(k * kTriThreads) + threadIdx.x;
        gt[k] = v.tile_off + (b.ty0 + (int)(q / b.ntx)) * v.tiles_x + b.tx0 + (int)(q % b.ntx);
        slot[k] = 0u;
        if (q < q1) slot[k] = FILL ? tile_start[tile_start_at(gt[k])] + pair_slot[a + q] : atomicAdd(&tile_count[gt[k]], 1u);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const unsigned q = q0 + (unsigned)(k * kTriThreads) + threadIdx.x;
        if (q >= q1) break;
        if (!FILL) {
            pair_slot[a + q] = slot[k];
        } else {
            bins[slot[k]] = tri;
            if (bin_pair) bin_pair[slot[k]] = a + q;
        }
    }
}

// Workgroups past the triangles' own: the listed large triangles.
// off(t): first pair of triangle t.
template <bool FILL, class Off>
__device__ __forceinline__ void bin_large(const ViewConst *__restrict__ views, const TriSetup *__restrict__ setup,
                                          unsigned capacity, int shift, int b, unsigned *__restrict__ tile_count,
                                          unsigned *__restrict__ pair_slot, const unsigned *__restrict__ tile_start,
                                          unsigned *__restrict__ bins, unsigned *__restrict__ bin_pair,
                                          const LargeLists &large, const DevCounters *counters, Off off) {
    for_large_items(large, counters, b, kLargeBlocks, [&](unsigned t) { return tile_box(setup[t], shift).n; },
                    [&](unsigned t, unsigned q0, unsigned n) {
                        const unsigned a = off(t);
                        if (a + n > capacity) return;                       // overflow path
                        const TriSetup &s = setup[t];
                        bin_range<FILL>(views[s.pad2[0]], s, t, a, q0, min(q0 + kLargeChunk, n), shift, tile_count,
                                        pair_slot, tile_start, bins, bin_pair);
                    });
}

// Silhouette mask of (view, triangle): oriented edge e is a silhouette when
// no triangle or more than one other triangle shares it, or when the
// neighbour across it faces the other way in this view.
__device__ __forceinline__ unsigned char silhouette_mask(const int *__restrict__ adj,
                                                         const signed char *__restrict__ facing_view, int t,
                                                         size_t face) {
    const int facing = facing_view[t];
    if (facing == 0) return 0;
    const bool sw = facing < 0;        // second and third vertex were exchanged
    const int nb[3] = {adj[3 * face], adj[3 * face + 1], adj[3 * face + 2]};
    unsigned mask = 0;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int a = (e + 1) % 3, b = (e + 2) % 3;
        const int oa = sw ? (a == 0 ? 0 : 3 - a) : a, ob = sw ? (b == 0 ? 0 : 3 - b) : b;
        const int o = 3 - oa - ob, n = o == 0 ? nb[0] : o == 1 ? nb[1] : nb[2];
        if (n < 0 || facing_view[n] != facing) mask |= 1u << e;
    }
    return (unsigned char)mask;
}

// Totals of the triangle passes' workgroups scanned in place by one workgroup,
// for plans with more than kMaxTriGroups groups of them.
__global__ __launch_bounds__(kTriThreads) void block_prefix_kernel(unsigned *__restrict__ total, int n) {
    __shared__ unsigned carry;
    const int tid = (int)threadIdx.x;
    if (tid == 0) carry = 0;
    for (int c = 0; c < n; c += 16 * kTriThreads) {
        unsigned v[16], o[16], sum;
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = c + k * kTriThreads + tid < n ? total[c + k * kTriThreads + tid] : 0u;
        tri_block_scan<16, true>(v, o, &sum);
        const unsigned base = carry;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (c + k * kTriThreads + tid < n) total[c + k * kTriThreads + tid] = add_sat(base, o[k]);
        if (tid == 0) {
            carry = add_sat(base, sum);
            if (c + 16 * kTriThreads >= n) total[n] = add_sat(base, sum);
        }
        __syncthreads();
    }
}

// Count pass.  A triangle's first pair is its offset in its workgroup plus the
// totals of the workgroups before, which every workgroup sums itself: the
// setup added them up by groups of kTriGroup, so that is a load or two a lane
// (a scan in a launch of its own before: 16 us for 24 views of 99k triangles).
// Past kMaxTriGroups groups it finds the totals scanned.  The silhouette masks ride along: they need every
// facing byte, as this pass needs every total.
//
// Bound by the latency of the tile counters' atomics, so a workgroup counts
// its own pairs first: where the tiles its triangles touch lie in a box of at
// most kTileTable tiles (the triangles of a mesh are neighbours), a table in
// LDS holds a counter for each of them, one global atomic per tile that has
// pairs fetches the tile's first slot, and a second walk over the pairs hands
// out the slots from the table.  Wider boxes (a strip across a large view,
// triangles in no order) aggregate a wave's equal tiles with ballots
// (wave_slot), which took the place of the table before: 64 scenes at 512^2
// 57 -> 32 us (36 with the group totals, but without a scan of 11), three
// 2048^2 maps and a 1080p view 43 -> 30, a 10k-triangle
// sphere at 512^2 20 -> 7 (no aggregation at all: 167, 159 and 9).  4096
// counters are 16 KB, so that eight workgroups share a CU, and all tiles of a
// 512^2 view.
constexpr int kTileTable = 4096;
__global__ __launch_bounds__(kTriThreads) void bin_count_kernel(
    const ViewConst *__restrict__ views, const TriBlock *__restrict__ blocks, int nblocks,
    const TriSetup *__restrict__ setup, const int *__restrict__ adj, const signed char *__restrict__ facing8,
    unsigned char *__restrict__ silm, const unsigned *__restrict__ pair_local,
    const unsigned *__restrict__ block_total, const unsigned long long *__restrict__ group_total, bool scanned,
    unsigned *__restrict__ pair_off, unsigned capacity, int shift,
    int ntri,
    unsigned *__restrict__ tile_count, unsigned *__restrict__ pair_slot, LargeLists large,
    unsigned *__restrict__ overflow_list, DevCounters *counters) {
    // the tile table, a wave's triangles, or the prefix of the groups' totals
    __shared__ union {
        unsigned table[kTileTable];
        BinWave wave[kTriThreads / 64];
        unsigned prefix[kMaxTriGroups];
    } sh;
    const int tid = (int)threadIdx.x;
    if ((int)blockIdx.x >= nblocks) {
        if (counters->large_len == 0) return;
        // the workgroup's own prefix of the groups' totals
        unsigned *prefix = sh.prefix;
        __shared__ unsigned carry;
        if (tid == 0) carry = 0;
        const int ngroups = (nblocks + kTriGroup - 1) / kTriGroup;
        for (int c = 0; c < ngroups && !scanned; c += kTriThreads) {
            const unsigned v[1] = {c + tid < ngroups ? word_sat(group_total[(c + tid) * kGroupStride]) : 0u};
            unsigned o[1], total;
            tri_block_scan<1, true>(v, o, &total);
            const unsigned base = carry;
            __syncthreads();
            if (c + tid < ngroups) prefix[c + tid] = add_sat(base, o[0]);
            if (tid == 0) carry = add_sat(base, total);
            __syncthreads();
        }
        bin_large<false>(views, setup, capacity, shift, (int)blockIdx.x - nblocks, tile_count, pair_slot, nullptr,
                         nullptr, nullptr, large, counters, [&](unsigned t) {
                             const ViewConst &v = views[setup[t].pad2[0]];
                             const int k = v.tri_block + (int)(t - v.setup_off) / kTriRun;
                             if (scanned) return min(add_sat(pair_local[t], block_total[k]), kPairEnd);
                             // in its group by each wave alone
                             unsigned before = 0;
                             for (int q = (k & ~(kTriGroup - 1)) + (tid & 63); q < k; q += 64) before = add_sat(before, block_total[q]);
#pragma unroll
                             for (int o = 32; o > 0; o >>= 1) before = add_sat(before, __shfl_xor(before, o, 64));
                             return min(add_sat(pair_local[t], add_sat(prefix[k / kTriGroup], before)), kPairEnd);
                         });
        return;
    }
    const TriBlock blk = blocks[blockIdx.x];
    const ViewConst &v = views[blk.view];
    const int t = blk.first + tid;
    const bool mine = t < v.nfaces;
    TileBox b{0, 0, 1, 0u};
    unsigned local = 0;
    if (mine) {
        b = tile_box(setup[v.setup_off + t], shift);
        local = pair_local[v.setup_off + t];
    }
    const int nty = (int)small_div(b.n, b.ntx);
    __shared__ unsigned part[kTriThreads / 64];
    __shared__ int boxes[kTriThreads / 64][4];        // the waves' tiles: first x, first y, last x, last y
    unsigned sum = 0;
    if (!scanned) {
        static_assert(kTriGroup <= kTriThreads, "a lane each");
        const int g = (int)blockIdx.x / kTriGroup;
        for (int k = tid; k < g; k += kTriThreads) sum = add_sat(sum, word_sat(group_total[k * kGroupStride]));
        if (g * kTriGroup + tid < (int)blockIdx.x) sum = add_sat(sum, block_total[g * kTriGroup + tid]);
    }
    const bool small = b.n > 0 && b.n <= kBigBin;
    int lo_x = small ? b.tx0 : 65536, lo_y = small ? b.ty0 : 65536;
    int hi_x = small ? b.tx0 + b.ntx - 1 : -1, hi_y = small ? b.ty0 + nty - 1 : -1;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sum = add_sat(sum, __shfl_xor(sum, o, 64));
        lo_x = min(lo_x, __shfl_xor(lo_x, o, 64));
        lo_y = min(lo_y, __shfl_xor(lo_y, o, 64));
        hi_x = max(hi_x, __shfl_xor(hi_x, o, 64));
        hi_y = max(hi_y, __shfl_xor(hi_y, o, 64));
    }
    if ((tid & 63) == 0) {
        int *q = boxes[tid >> 6];
        part[tid >> 6] = sum;
        q[0] = lo_x;
        q[1] = lo_y;
        q[2] = hi_x;
        q[3] = hi_y;
    }
    __syncthreads();
    const unsigned base =
        scanned ? block_total[blockIdx.x] : add_sat(add_sat(part[0], part[1]), add_sat(part[2], part[3]));
#pragma unroll
    for (int k = 0; k < kTriThreads / 64; ++k) {
        lo_x = min(lo_x, boxes[k][0]);
        lo_y = min(lo_y, boxes[k][1]);
        hi_x = max(hi_x, boxes[k][2]);
        hi_y = max(hi_y, boxes[k][3]);
    }
    const int bw = hi_x - lo_x + 1, nbox = hi_x < 0 ? 0 : bw * (hi_y - lo_y + 1);
    const bool table = nbox <= kTileTable;            // the same in every lane
    if (table)
        for (int k = tid; k < nbox; k += kTriThreads) sh.table[k] = 0u;
    if ((int)blockIdx.x == nblocks - 1 && tid == 0) {
        const unsigned total = min(scanned ? block_total[nblocks] : add_sat(base, block_total[blockIdx.x]), kPairEnd);
        pair_off[ntri] = total;
        unsigned long long all = total;                      // for the plan's statistics
        if (total == kPairEnd) {
            all = 0;
            for (int g = 0; g < nblocks; g += kTriGroup) all += group_total[g / kTriGroup * kGroupStride];
        }
        counters->pairs = all;
    }
    unsigned cnt = 0;
    BinItem it{};
    it.a = min(add_sat(local, base), kPairEnd);
    it.ntx = b.ntx;
    it.tile0 = v.tile_off + b.ty0 * v.tiles_x + b.tx0;
    if (mine) {
        const int si = v.setup_off + t;
        pair_off[si] = it.a;
        const unsigned end = it.a + b.n;                     // at most kPairEnd and a view's tiles: no wrap
        if (end > capacity) {                                // overflow path
            if (b.n) overflow_list[atomicAdd(&counters->overflow_list_len, 1u)] = (unsigned)si;
        } else if (small) {
            cnt = b.n;
        }
        silm[si] = silhouette_mask(adj, facing8 + v.setup_off, t, (size_t)(v.face_off + t));
    }
    if (table) {
        if (nbox == 0) return;
        unsigned *first = sh.table + (b.ty0 - lo_y) * bw + (b.tx0 - lo_x);
        __syncthreads();
        if (cnt)
            for (int y = 0; y < nty; ++y)
                for (int x = 0; x < b.ntx; ++x) atomicAdd(first + y * bw + x, 1u);
        __syncthreads();
        const int tile0 = v.tile_off + lo_y * v.tiles_x + lo_x;
        for (int c = tid; c < nbox; c += kTriThreads * kPairSteps) {
            unsigned n[kPairSteps];
#pragma unroll
            for (int u = 0; u < kPairSteps; ++u) {
                const int k = c + u * kTriThreads;
                n[u] = k < nbox ? sh.table[k] : 0u;
                if (n[u]) n[u] = atomicAdd(&tile_count[tile0 + (k / bw) * v.tiles_x + k % bw], n[u]);
            }
#pragma unroll
            for (int u = 0; u < kPairSteps; ++u)
                if (c + u * kTriThreads < nbox) sh.table[c + u * kTriThreads] = n[u];
        }
        __syncthreads();
        if (cnt) {
            unsigned *slot = pair_slot + it.a;
            for (int y = 0; y < nty; ++y)
                for (int x = 0; x < b.ntx; ++x) *slot++ = atomicAdd(first + y * bw + x, 1u);
        }
        return;
    }
    for_wave_pairs(sh.wave[tid >> 6], cnt, it,
                   [&](int n, const BinItem (&b)[kPairSteps], const unsigned (&q)[kPairSteps],
                       const bool (&has)[kPairSteps], const int (&starts)[kPairSteps]) {
                       WaveSlot s[kPairSteps];
                       unsigned base[kPairSteps];
#pragma unroll
                       for (int u = 0; u < kPairSteps; ++u) {
                           base[u] = 0u;
                           if (u >= n) continue;
                           const unsigned r = small_div(q[u], b[u].ntx);
                           const int gt = has[u] ? b[u].tile0 + (int)r * v.tiles_x + (int)(q[u] - r * (unsigned)b[u].ntx) : 0;
                           s[u] = wave_slot(has[u], gt, starts[u] > 8);
                           if (s[u].size) base[u] = atomicAdd(&tile_count[gt], s[u].size);
                       }
#pragma unroll
                       for (int u = 0; u < kPairSteps; ++u)
                           if (u < n) {
                               const unsigned slot = (unsigned)__shfl((int)base[u], s[u].leader, 64) + s[u].rank;
                               if (has[u]) pair_slot[b[u].a + q[u]] = slot;
                           }
                   });
}

// Fill pass.  With overflowed triangles, the workgroups also clear the keys,
// which the raster then minimizes into (raster_kernel).
__global__ __launch_bounds__(kTriThreads) void bin_fill_kernel(
    const ViewConst *__restrict__ views, const TriBlock *__restrict__ blocks, int nblocks,
    const TriSetup *__restrict__ setup, const unsigned *__restrict__ pair_off, unsigned capacity, int shift,
    unsigned *__restrict__ pair_slot, const unsigned *__restrict__ tile_start, unsigned *__restrict__ bins,
    unsigned *__restrict__ bin_pair, LargeLists large, const DevCounters *counters,
    unsigned long long *__restrict__ keys, long long nkeys) {
    __shared__ BinWave wave[kTriThreads / 64];
    const int tid = (int)threadIdx.x;
    if (counters->overflow_list_len)
        for (long long i = (long long)blockIdx.x * kTriThreads + tid; i < nkeys; i += (long long)gridDim.x * kTriThreads)
            keys[i] = kBgKey;
    if ((int)blockIdx.x >= nblocks) {
        bin_large<true>(views, setup, capacity, shift, (int)blockIdx.x - nblocks, nullptr, pair_slot, tile_start, bins,
                        bin_pair, large, counters, [&](unsigned t) { return pair_off[t]; });
        return;
    }
    const TriBlock blk = blocks[blockIdx.x];
    const ViewConst &v = views[blk.view];
    const int t = blk.first + tid;
    unsigned cnt = 0;
    BinItem it{};
    if (t < v.nfaces) {
        const int si = v.setup_off + t;
        const TileBox b = tile_box(setup[si], shift);
        it.a = pair_off[si];
        it.ntx = b.ntx;
        it.tile0 = v.tile_off + b.ty0 * v.tiles_x + b.tx0;
        it.tri = (unsigned)si;
        if (it.a + b.n <= capacity && b.n <= kBigBin) cnt = b.n;
    }
    for_wave_pairs(wave[tid >> 6], cnt, it,
                   [&](int n, const BinItem (&b)[kPairSteps], const unsigned (&q)[kPairSteps],
                       const bool (&has)[kPairSteps], const int (&starts)[kPairSteps]) {
                       unsigned pos[kPairSteps];
#pragma unroll
                       for (int u = 0; u < kPairSteps; ++u) {
                           pos[u] = 0u;
                           if (u >= n || !has[u]) continue;
                           const unsigned r = small_div(q[u], b[u].ntx);
                           const int gt = b[u].tile0 + (int)r * v.tiles_x + (int)(q[u] - r * (unsigned)b[u].ntx);
                           pos[u] = tile_start[tile_start_at(gt)] + pair_slot[b[u].a + q[u]];
                       }
#pragma unroll
                       for (int u = 0; u < kPairSteps; ++u)
                           if (u < n && has[u]) {
                               bins[pos[u]] = b[u].tri;
                               if (bin_pair) bin_pair[pos[u]] = b[u].a + q[u];
                           }
                   });
}

// Tile starts: a workgroup scans kScanBlock tiles' counts and takes its base
// from the running total, so one launch does all of them (which block comes
// first in the bins does not matter).
__global__ __launch_bounds__(kTriThreads) void tile_scan_kernel(const unsigned *__restrict__ count,
                                                                unsigned *__restrict__ start, int ntiles,
                                                                DevCounters *counters) {
    constexpr int PER = kScanBlock / kTriThreads;
    const int t0 = blockIdx.x * kScanBlock;
    unsigned v[PER], off[PER], total;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int t = t0 + k * kTriThreads + (int)threadIdx.x;
        v[k] = t < ntiles ? count[t] : 0u;
    }
    tri_block_scan(v, off, &total);
    __shared__ unsigned base;
    if (threadIdx.x == 0) {
        base = atomicAdd(&counters->bin_cursor, total);
        start[tile_start_at(t0) + min(kScanBlock, ntiles - t0)] = base + total;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int t = t0 + k * kTriThreads + (int)threadIdx.x;
        if (t < ntiles) start[tile_start_at(t)] = base + off[k];
    }
}

// ----------------------------------------------------------------------------- raster

// Triangles that did not fit the bins: workgroup b of kOverflowBlocks takes
// every kOverflowBlocks-th of the list, with an atomic minimum per covered
// sample.  They run in the tile groups' launch; their keys and the groups'
// meet in the same atomic minimum.  The first thread also adds the list's
// length to the overflow count.
constexpr int kOverflowBlocks = 512;
__device__ __forceinline__ void overflow_raster(const ViewConst *__restrict__ views, const TriSetup *__restrict__ setup,
                                                const unsigned *__restrict__ list, unsigned n, unsigned b,
                                                DevCounters *counters, unsigned long long *__restrict__ keys) {
    if (n && b == 0 && threadIdx.x == 0) counters->overflow += n;
    for (unsigned o = b; o < n; o += kOverflowBlocks) {
        const unsigned si = list[o];
        const TriSetup &s = setup[si];
        const ViewConst &v = views[s.pad2[0]];
        const RasterTri r = load_raster_tri(s, si - (unsigned)v.setup_off, 0, 0);
        const int w = s.bx1 - s.bx0 + 1, h = s.by1 - s.by0 + 1;
        if (w <= 0 || h <= 0) continue;
        const long long npix = (long long)w * h;
        for (long long q = threadIdx.x; q < npix; q += blockDim.x) {
            const int i = s.bx0 + (int)(q % w), j = s.by0 + (int)(q / w);
            const unsigned long long key = pixel_key(r, sample_pos(i), sample_pos(j));
            if (key != kBgKey) atomicMin(&keys[v.pix_off + (long long)j * v.W + i], key);
        }
    }
}

// One workgroup rasterizes a group of kGroup consecutive tiles of the global
// tile list, whose bins are one contiguous range of entries.  The range
// streams through the workgroup's lanes, an entry a lane: the lane reads the
// triangle's record and clips its bounding box to its tile.  A triangle with
// few samples there is tested by its lane alone, sample by sample, stepping
// the edge functions; the others go to a list in LDS that the four waves
// share, 64 samples of a triangle at a time.  Both take the minimum of the
// samples' keys in LDS, so neither the order of the entries nor the split
// matters.  What bounds it: the records' loads and the tests.  A mesh of
// pixel-sized triangles keeps every lane on a triangle of its own (the
// wave-wide test alone uses 64 lanes on the four samples of a 2 x 2 box), a
// crowded tile is shared by four waves, and a group of nearly empty tiles
// waits for one chain of loads instead of one per tile.  Against one wave per
// tile testing its bin an entry at a time: 64 scenes at 512^2 388 -> 211 us,
// 8 x 1024^2 maps and 16 views of a 99k-triangle sphere 432 -> 102, four
// scenes at 200^2 (hundreds of entries a tile) 133 -> 24.  Groups of 4 or 16
// tiles: 338 and 313 us on the 64 scenes where 8 took 259; 6 waves per SIMD 271,
// 8 (spills) 403.
constexpr int kRasterThreads = 256;
// Groups are cheap over sky and dear over a mesh, so the XCDs take turns of
// kGroupRun of them (an odd number, so that a turn does not repeat with the rows
// of a view) instead of a range each: 64 scenes 259 -> 211 us (16: 231, 5: 238,
// 128: 303), 24 views of 99k triangles 142 -> 102, 28,600 groups of a 1080p view
// and its maps 163 -> 140.  In a few rounds of resident workgroups (1,792 at a
// time) there is less to even out, and the ranges stay for the records that
// neighbours share: 7,164 groups of a 960 x 540 view and its maps 52 us, in turns
// 58.  The line lies between that and the smallest grid measured faster in turns
// (24,576 groups).
constexpr int kGroupRun = 23, kRangeGroups = 8192;
constexpr int kWide = 128;      // records of the shared list; a chunk with more takes another round

template <int T>
struct RasterShape {
    static constexpr int kGroup = T == 8 ? 8 : T == 16 ? 2 : 1;     // tiles per workgroup
    static constexpr int kPix = kGroup * T * T;
};

template <int T>
__global__ __launch_bounds__(kRasterThreads) __attribute__((amdgpu_waves_per_eu(T == 8 ? 7 : 4))) void raster_kernel(
    const ViewConst *__restrict__ views, const int *__restrict__ tile_view, int ntiles,
    const TriSetup *__restrict__ setup, const unsigned *__restrict__ tile_start, const unsigned *__restrict__ bins,
    unsigned long long *__restrict__ keys, const unsigned *__restrict__ overflow_list, DevCounters *counters,
    int ngroups) {
    using RS = RasterShape<T>;
    constexpr int G = RS::kGroup;
    const unsigned nover = counters->overflow_list_len;
    if ((int)blockIdx.x >= ngroups) {
        overflow_raster(views, setup, overflow_list, nover, (unsigned)((int)blockIdx.x - ngroups), counters, keys);
        return;
    }
    struct TileInfo {
        long long pix;           // key index of the tile's first sample
        int x0, y0, W, H, setup_off;
    };
    __shared__ unsigned long long best[RS::kPix];
    __shared__ TileInfo info[G];
    __shared__ __align__(16) RasterTri wide[kWide];
    __shared__ unsigned nwide;
    const int gb = (int)blockIdx.x;
    const int g0 = (ngroups > kRangeGroups ? xcd_turns<kGroupRun>(gb, ngroups) : xcd_remap(gb, ngroups)) * G;
    const int ng = min(G, ntiles - g0);
    const int tid = (int)threadIdx.x, lane = tid & 63;
    unsigned ts[G + 1];
#pragma unroll
    for (int k = 0; k <= G; ++k) ts[k] = tile_start[tile_start_at(g0) + min(k, ng)];     // kScanBlock is whole groups
    // the first entry's record is requested before anything waits
    unsigned e = ts[0] + (unsigned)tid;
    unsigned si = 0;
    TriSetup st;
    if (e < ts[G]) {
        si = bins[e];
        st = setup[si];
    }
    if (tid < ng) {
        const ViewConst &v = views[tile_view[g0 + tid]];
        const int lt = g0 + tid - v.tile_off;
        TileInfo ti;
        ti.x0 = (lt % v.tiles_x) * T;
        ti.y0 = (lt / v.tiles_x) * T;
        ti.W = v.W;
        ti.H = v.H;
        ti.pix = v.pix_off + (long long)ti.y0 * v.W + ti.x0;
        ti.setup_off = v.setup_off;
        info[tid] = ti;
    }
#pragma unroll
    for (int q = tid; q < RS::kPix; q += kRasterThreads) best[q] = kBgKey;
    if (tid == 0) nwide = 0u;
    __syncthreads();
    for (unsigned c = ts[0]; c < ts[G]; c += kRasterThreads) {          // uniform
        RasterTri r;
        int area = 0, x0 = 0, x1 = 0, y0 = 0, y1 = 0, k = 0;
        if (e < ts[G]) {
#pragma unroll
            for (int q = 1; q < G; ++q) k += e >= ts[q] ? 1 : 0;
            const int ox = info[k].x0, oy = info[k].y0;
            r = load_raster_tri(st, si - (unsigned)info[k].setup_off, ox, oy);
            x0 = max((int)st.bx0 - ox, 0);
            x1 = min((int)st.bx1 - ox, T - 1);
            y0 = max((int)st.by0 - oy, 0);
            y1 = min((int)st.by1 - oy, T - 1);
            area = touches(r, x0, x1, y0, y1) ? (x1 - x0 + 1) * (y1 - y0 + 1) : 0;
            r.box |= (unsigned)x0 | (unsigned)x1 << 5 | (unsigned)y0 << 10 | (unsigned)y1 << 15 | (unsigned)k << 20;
        }
        // largest box that a lane tests alone: each step up costs the wave
        // that many more samples and saves one wave-wide test per triangle
        const int n0 = __popcll(__ballot(area > 0)), n16 = __popcll(__ballot(area > 16)),
                  n32 = __popcll(__ballot(area > 32)), n64 = __popcll(__ballot(area > 64));
        const int most = n16 - n64 > 48 ? 64 : n16 - n32 > 16 ? 32 : n0 - n16 > 8 ? 16 : 0;
        const bool own = area > 0 && area <= most, shared = area > most;
        const unsigned long long m = __ballot(shared);
        unsigned at = ~0u;                    // this lane's place in the list
        if (m) {
            unsigned first = 0;
            if (lane == 0) first = atomicAdd(&nwide, (unsigned)__popcll(m));
            first = (unsigned)__builtin_amdgcn_readfirstlane((int)first);
            if (shared) at = first + (unsigned)__popcll(m & ((1ull << lane) - 1ull));
            if (at < kWide) wide[at] = r;
        }
        if (own)
            step_box<T>(r, x0, x1, y0, area, best + k * (T * T) + y0 * T,
                        [](unsigned long long *p, unsigned long long key) { atomicMin(p, key); });
        __syncthreads();
        const int n = (int)nwide;
        for (int base = 0; base < n; base += kWide) {                   // uniform
            if (base > 0) {
                __syncthreads();
                if (at != ~0u && at >= (unsigned)base && at < (unsigned)(base + kWide)) wide[at - base] = r;
                __syncthreads();
            }
            for (int j = tid >> 6; j < min(n - base, kWide); j += kRasterThreads / 64) {
                const RasterTri w = wide[j];
                const int wx0 = w.box & 31, wx1 = (w.box >> 5) & 31, wy0 = (w.box >> 10) & 31, wy1 = (w.box >> 15) & 31;
                unsigned long long *tb = best + ((w.box >> 20) & 15) * (T * T);
                // the tile's 8 x 8 blocks that the bounding box touches
                if constexpr (T == 8) {
                    const int lx = lane & 7, ly = lane >> 3;
                    if (lx >= wx0 && lx <= wx1 && ly >= wy0 && ly <= wy1) {
                        const unsigned long long key = pixel_key(w, sample_pos(lx), sample_pos(ly));
                        if (key != kBgKey) atomicMin(&tb[lane], key);
                    }
                    continue;
                }
                for (int by = wy0 >> 3; by <= wy1 >> 3; ++by)
                    for (int bx = wx0 >> 3; bx <= wx1 >> 3; ++bx) {
                        const int lx = bx * 8 + (lane & 7), ly = by * 8 + (lane >> 3);
                        if (lx < wx0 || lx > wx1 || ly < wy0 || ly > wy1) continue;
                        const unsigned long long key = pixel_key(w, sample_pos(lx), sample_pos(ly));
                        if (key != kBgKey) atomicMin(&tb[ly * T + lx], key);
                    }
            }
        }
        __syncthreads();
        if (c + kRasterThreads < ts[G]) {
            if (tid == 0) nwide = 0u;
            e += kRasterThreads;
            if (e < ts[G]) {
                si = bins[e];
                st = setup[si];
            }
            __syncthreads();
        }
    }
    // store the group as rows of its tiles side by side
#pragma unroll
    for (int q = tid; q < RS::kPix; q += kRasterThreads) {
        const int row = q / (G * T), col = q % (G * T), k = col / T, lx = col % T;
        if (k >= ng) continue;
        const TileInfo &ti = info[k];
        if (!(ti.x0 + lx < ti.W && ti.y0 + row < ti.H)) continue;
        unsigned long long *key = keys + ti.pix + (long long)row * ti.W + lx;
        const unsigned long long m = best[k * (T * T) + row * T + lx];
        if (nover == 0) *key = m;
        else if (m != kBgKey) atomicMin(key, m);       // with the overflowed triangles; the fill pass cleared the keys
    }
}

// ----------------------------------------------------------------------------- host launchers

hipError_t launch_light_frames(ViewConst *views, const CamStatic *cams, const float *params, int L, float *jac,
                               float *zc_out, void *z1, size_t bytes1, void *z2, size_t bytes2, const ClearRows &rows,
                               hipStream_t s) {
    const int nf = (L + 63) / 64;
    const size_t n1 = bytes1 / 4, n2 = bytes2 / 4;
    const size_t nz = std::min<size_t>((n1 + n2 + 255) / 256, 16384);
    if (nf + nz == 0) return hipSuccess;
    hipLaunchKernelGGL(light_frames_kernel, dim3((unsigned)(nf + nz)), dim3(64), 0, s, views, cams, params, L, zc_out,
                       jac, nf, (unsigned *)z1, n1, (unsigned *)z2, n2, rows);
    return hipGetLastError();
}

hipError_t launch_setup(const ViewConst *views, const TriBlock *blocks, int nblocks, const int *faces,
                        const float *verts, const float *albedo, int C, TriVerts *tv, TriSetup *setup,
                        signed char *facing8, unsigned *pair_local, unsigned *block_total,
                        unsigned long long *group_total, const LargeLists &large, int tile, DevCounters *counters,
                        hipStream_t s) {
    if (nblocks == 0) return hipSuccess;
    hipLaunchKernelGGL(setup_kernel, dim3(nblocks), dim3(kTriThreads), 0, s, views, blocks, faces, verts, albedo, C, tv,
                       setup, facing8, pair_local, block_total, group_total, large, __builtin_ctz(tile), counters);
    return hipGetLastError();
}

hipError_t launch_binning(const ViewConst *views, const TriBlock *blocks, int nblocks, const TriSetup *setup,
                          const int *adj, const signed char *facing8, unsigned char *silm, const unsigned *pair_local,
                          unsigned *block_total, const unsigned long long *group_total, unsigned *pair_off,
                          int ntri, unsigned capacity, int tile,
                          unsigned *tile_count, unsigned *tile_start, unsigned *pair_slot, int ntiles, unsigned *bins,
                          unsigned *bin_pair, unsigned *overflow_list, const LargeLists &large,
                          DevCounters *counters, unsigned long long *keys, long long nkeys,
                          hipStream_t s) {
    if (ntri > kScanBlock * kScanBlock || ntiles > kScanBlock * kScanBlock) return hipErrorInvalidValue;
    const bool scanned = nblocks > kTriGroup * kMaxTriGroups;
    if (scanned) hipLaunchKernelGGL(block_prefix_kernel, dim3(1), dim3(kTriThreads), 0, s, block_total, nblocks);
    const dim3 grid(nblocks + kLargeBlocks);
    const int shift = __builtin_ctz(tile);
    if (nblocks > 0)
        hipLaunchKernelGGL(bin_count_kernel, grid, dim3(kTriThreads), 0, s, views, blocks, nblocks, setup, adj, facing8,
                           silm, pair_local, block_total, group_total, scanned, pair_off, capacity, shift, ntri, tile_count,
                           pair_slot, large, overflow_list, counters);
    if (ntiles > 0)
        hipLaunchKernelGGL(tile_scan_kernel, dim3((ntiles + kScanBlock - 1) / kScanBlock), dim3(kTriThreads), 0, s,
                           tile_count, tile_start, ntiles, counters);
    if (nblocks > 0)
        hipLaunchKernelGGL(bin_fill_kernel, grid, dim3(kTriThreads), 0, s, views, blocks, nblocks, setup, pair_off,
                           capacity, shift, pair_slot, tile_start, bins, bin_pair, large, counters, keys,
                           nkeys);
    return hipGetLastError();
}

hipError_t launch_raster(const ViewConst *views, const int *tile_view, int ntiles, int tile, const TriSetup *setup,
                         const unsigned *tile_start, const unsigned *bins, const unsigned *overflow_list,
                         DevCounters *counters, unsigned long long *keys, hipStream_t s) {
    if (ntiles == 0) return hipSuccess;
#define DSM_RASTER(TT)                                                                                              \
    do {                                                                                                            \
        const int groups = (ntiles + RasterShape<TT>::kGroup - 1) / RasterShape<TT>::kGroup;                       \
        hipLaunchKernelGGL(raster_kernel<TT>, dim3(groups + kOverflowBlocks), dim3(kRasterThreads), 0, s, views,   \
                           tile_view, ntiles, setup, tile_start, bins, keys, overflow_list, counters, groups);     \
    } while (0)
    if (tile == 8) DSM_RASTER(8);
    else if (tile == 16) DSM_RASTER(16);
    else DSM_RASTER(32);
#undef DSM_RASTER
    return hipGetLastError();
}

}  // namespace dsm
