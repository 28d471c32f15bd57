// Edge antialiasing at primitive borders, shared by the light view (the
// smoothed shadow map f~, f^2~ of Sec. 4, which Alg. 1 filters) and the
// camera view (the shaded image).
//
// For two horizontally or vertically adjacent samples owned by different
// triangles: the sample with the smaller depth|id key is the front sample F,
// the other O.  The front triangle's edges whose edge function is negative at
// O are exit edges; the first one crossed on the way F -> O (smallest
// float32 ratio E(F) / (E(F) - E(O)), lower edge index on ties) is taken.
// The pair is smoothed only if that edge is a silhouette in the view
// (boundary, non-manifold, or neighbour of opposite facing; precomputed per
// triangle as a byte per view, silhouette_mask) and, so that
// each edge is handled in one direction only, |dY| > |dX| for horizontal
// pairs and |dY| <= |dX| for vertical ones.  The continuous crossing
// alpha = E(F) / (E(F) - E(O)) is computed from the unsnapped vertex
// positions (float64): alpha > 1/2 moves O toward F by (alpha - 1/2),
// otherwise F moves toward O by (1/2 - alpha).  Deltas use pre-smoothing
// values; every sample gathers the deltas of its four pairs.
#pragma once

#include "dsm_internal.h"

namespace dsm {

__device__ __forceinline__ long long aa_edge_fn(int xa, int ya, int xb, int yb, int px, int py) {
    return (long long)(xb - xa) * (py - ya) - (long long)(yb - ya) * (px - xa);
}

struct AAPair {
    int recv;          // 0: receiver is the front sample, 1: the other sample
    float w;           // blend weight |alpha - 1/2|
    int va, vb;        // scene-local vertex indices of the chosen edge
    double alpha;      // continuous crossing
    // partial derivatives of alpha w.r.t. the clip coordinates (x, y, w) of va and vb
    double dax, day, daw, dbx, dby, dbw;
};

__device__ __forceinline__ int orig_slot(int s, bool swapped) { return swapped ? (s == 0 ? 0 : 3 - s) : s; }

__device__ __forceinline__ void clip_f64(const float *M, const float *p, double c[4]) {
    const double x = p[0], y = p[1], z = p[2];
    for (int r = 0; r < 4; ++r) c[r] = ((double)M[4 * r] * x + (double)M[4 * r + 1] * y) + (double)M[4 * r + 2] * z +
                                     (double)M[4 * r + 3];
}

// Evaluate the pair (self sample s, neighbour sample n) whose front triangle
// is t (self_is_front: the self sample's).  Returns false when the pair is not
// smoothed.
template <bool WANT_GRAD>
__device__ __forceinline__ bool aa_eval(const ViewConst &v, const TriSetup *__restrict__ setup,
                                        const int *__restrict__ faces, const unsigned char *__restrict__ silm,
                                        const float *__restrict__ verts, unsigned t, bool self_is_front, int is,
                                        int js, int in_, int jn, bool horiz, AAPair &out) {
    const int fi = self_is_front ? is : in_, fj = self_is_front ? js : jn;
    const int oi = self_is_front ? in_ : is, oj = self_is_front ? jn : js;
    const unsigned sm = silm[v.setup_off + t];
    const TriSetup &S = setup[v.setup_off + t];
    // the triangle's three vertex indices, loaded with its setup record so
    // that the vertex fetch below is the only load that waits on the edge choice
    const size_t fidx = (size_t)(v.face_off + (int)t);
    const int fv[3] = {faces[3 * fidx], faces[3 * fidx + 1], faces[3 * fidx + 2]};
    const int fX = fi * kSub + kSub / 2, fY = fj * kSub + kSub / 2;
    const int oX = oi * kSub + kSub / 2, oY = oj * kSub + kSub / 2;
    float best = 0.f;
    int ebest = -1;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int a = (e + 1) % 3, b = (e + 2) % 3;
        const long long eo = aa_edge_fn(S.X[a], S.Y[a], S.X[b], S.Y[b], oX, oY);
        if (eo < 0) {
            const long long ef = aa_edge_fn(S.X[a], S.Y[a], S.X[b], S.Y[b], fX, fY);
            const float r = (float)(double)ef / (float)(double)(ef - eo);
            if (ebest < 0 || r < best) { best = r; ebest = e; }
        }
    }
    if (ebest < 0) return false;
    const int a = (ebest + 1) % 3, b = (ebest + 2) % 3;
    const int dX = S.X[b] - S.X[a], dY = S.Y[b] - S.Y[a];
    const bool dir_ok = horiz ? (abs(dY) > abs(dX)) : (abs(dY) <= abs(dX));
    if (!dir_ok) return false;
    if (!((sm >> ebest) & 1)) return false;
    const bool sw = S.swapped != 0;
    const int oa = orig_slot(a, sw), ob = orig_slot(b, sw);
    out.va = oa == 0 ? fv[0] : oa == 1 ? fv[1] : fv[2];
    out.vb = ob == 0 ? fv[0] : ob == 1 ? fv[1] : fv[2];
    double ca[4], cb[4];
    clip_f64(v.M, verts + 3 * (size_t)(v.vert_off + out.va), ca);
    clip_f64(v.M, verts + 3 * (size_t)(v.vert_off + out.vb), cb);
    const double hw = 0.5 * v.W, hh = 0.5 * v.H;
    const double xa = (ca[0] / ca[3] + 1.0) * hw, ya = (1.0 - ca[1] / ca[3]) * hh;
    const double xb = (cb[0] / cb[3] + 1.0) * hw, yb = (1.0 - cb[1] / cb[3]) * hh;
    const double pfx = fi + 0.5, pfy = fj + 0.5, pox = oi + 0.5, poy = oj + 0.5;
    const double eF = (xb - xa) * (pfy - ya) - (yb - ya) * (pfx - xa);
    const double eO = (xb - xa) * (poy - ya) - (yb - ya) * (pox - xa);
    const double D = eF - eO;
    const double alpha = eF / D;
    out.alpha = alpha;
    if (alpha > 0.5) {
        out.recv = 1;
        out.w = (float)(alpha - 0.5);
    } else {
        out.recv = 0;
        out.w = (float)(0.5 - alpha);
    }
    if (WANT_GRAD) {
        // gradient terms only: one reciprocal each of D^2 and of the two w
        const double rD = 1.0 / (D * D), ra = 1.0 / ca[3], rb = 1.0 / cb[3];
        const double dF = -eO * rD, dO = eF * rD;    // d alpha / d eF, d alpha / d eO
        // d E(p) / d (xa, ya, xb, yb)
        const double gxa = (dF * (yb - pfy) + dO * (yb - poy)) * hw;
        const double gya = (dF * (pfx - xb) + dO * (pox - xb)) * hh;
        const double gxb = (dF * (pfy - ya) + dO * (poy - ya)) * hw;
        const double gyb = (-dF * (pfx - xa) - dO * (pox - xa)) * hh;
        // screen coordinates to clip (x, y, w)
        out.dax = gxa * ra;
        out.day = -gya * ra;
        out.daw = (gya * ca[1] - gxa * ca[0]) * (ra * ra);
        out.dbx = gxb * rb;
        out.dby = -gyb * rb;
        out.dbw = (gyb * cb[1] - gxb * cb[0]) * (rb * rb);
    }
    return true;
}

// Which of sample (i, j)'s pairs with its four neighbours (order -x, +x, -y, +y)
// can be smoothed at all: different triangles and a front triangle with a
// silhouette edge in this view.  All neighbour keys are loaded together, then
// all silhouette bytes, so a sample waits for two dependent loads instead of
// two per neighbour (one when no lane of its wave has a differing neighbour).
// The view must have faces.
__device__ __forceinline__ void aa_candidates(const ViewConst &v, const unsigned long long *__restrict__ kv,
                                              const unsigned char *__restrict__ silm, unsigned long long ks, int i,
                                              int j, bool (&cand)[4]) {
    unsigned long long kn[4];
    bool inb[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int in_ = i + (d == 0 ? -1 : d == 1 ? 1 : 0), jn = j + (d == 2 ? -1 : d == 3 ? 1 : 0);
        inb[d] = in_ >= 0 && in_ < v.W && jn >= 0 && jn < v.H;
        kn[d] = kv[inb[d] ? jn * v.W + in_ : j * v.W + i];
    }
    bool differ[4], any = false;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        differ[d] = inb[d] && (unsigned)kn[d] != (unsigned)ks;
        any = any || differ[d];
        cand[d] = false;
    }
    // a wave inside one triangle (most of a ground plane) waits for no
    // silhouette byte at all
    if (__ballot(any) != 0ull) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const unsigned front = ks < kn[d] ? (unsigned)ks : (unsigned)kn[d];
            const unsigned char sil = differ[d] ? silm[v.setup_off + front] : (unsigned char)0;
            cand[d] = differ[d] && sil != 0;
        }
    }
}

// Smoothing of a region of kAaW x kAaH samples by one wave: a lane owns a
// column of kAaH samples.  Every pair of neighbours with at least one sample
// in the region has a slot: the pair of columns c - 1 and c of row r (c = 0..64)
// at r * 65 + c, the pair of rows r - 1 and r of column c (r = 0..4) at
// 260 + r * 64 + c; its sample a is the left or upper one, b the other.
//
// A pair is a candidate when its triangles differ and the front one has a
// silhouette edge in this view.  Candidates are rare and cost three dependent
// loads and some 200 instructions, many in float64.  They are therefore
// listed and evaluated a pair a lane, each pair once for both of its samples
// (a pair across a region's border once in each region), and the result goes
// to the pair's slot, so a sample adds its pairs' terms in the order
// -x, +x, -y, +y whichever lane evaluated them.  The keys of a column are
// loaded once (six per four samples; the horizontal neighbours' keys come
// from the lanes beside), the silhouette bytes once per pair.
constexpr int kAaW = 64, kAaH = 4;
constexpr int kAaRow = kAaW + 1, kAaVert = kAaH * kAaRow, kAaSlots = kAaVert + (kAaH + 1) * kAaW;

constexpr unsigned char kAaB = 1, kAaA = 2, kAaCand = 4;    // b receives, a receives, candidate

struct AARegion {
    unsigned short item[kAaSlots];     // listed slots
    unsigned char state[kAaSlots];
    float w[kAaSlots];                 // blend weights
};

__host__ __device__ __forceinline__ int aa_regions(int W, int H) {
    return ((W + kAaW - 1) / kAaW) * ((H + kAaH - 1) / kAaH);
}

__device__ __forceinline__ unsigned long long shfl_key(unsigned long long k, int src) {
    const unsigned lo = (unsigned)__shfl((int)(unsigned)k, src, 64), hi = (unsigned)__shfl((int)(unsigned)(k >> 32), src, 64);
    return (unsigned long long)hi << 32 | lo;
}

// Keys of the region's column i = i0 + lane: k[r] of row j0 - 1 + r, and of
// the sample beside the region's edge columns (lane 0: left, lane 63: right)
// in rows j0 .. j0 + 3.
struct AAKeys {
    unsigned long long k[kAaH + 2], side[kAaH];
    bool ok[kAaH + 2], side_ok[kAaH];
};

__device__ __forceinline__ AAKeys aa_keys(const unsigned long long *__restrict__ kv, int W, int H, int i0, int j0,
                                          int lane) {
    AAKeys r;
    const int i = i0 + lane, is = lane == 0 ? i - 1 : i + 1;
    const bool col = i < W, edge = (lane == 0 && i > 0) || (lane == 63 && is < W);
#pragma unroll
    for (int q = 0; q < kAaH + 2; ++q) {
        const int j = j0 - 1 + q;
        r.ok[q] = col && j >= 0 && j < H;
        r.k[q] = r.ok[q] ? kv[j * W + i] : kBgKey;
    }
#pragma unroll
    for (int q = 0; q < kAaH; ++q) {
        r.side_ok[q] = edge && r.ok[q + 1];
        r.side[q] = r.side_ok[q] ? kv[(j0 + q) * W + is] : kBgKey;
    }
    return r;
}

// List the region's candidate pairs; returns their number (uniform).  When
// it is not zero, state[] holds kAaCand for candidates and 0 elsewhere.  All
// lanes of the (one-wave) workgroup call.
__device__ __forceinline__ int aa_list(AARegion &g, const AAKeys &k, const unsigned char *__restrict__ sil, int lane) {
    // left pair and (lane 63) right pair of each row, upper pair of each row and of the row below
    unsigned front[2 * kAaH + kAaH + 1];
    bool differ[2 * kAaH + kAaH + 1];
    bool any = false;
#pragma unroll
    for (int q = 0; q < kAaH; ++q) {
        const unsigned long long up = shfl_key(k.k[q + 1], lane - 1);
        const bool up_ok = __shfl((int)k.ok[q + 1], lane - 1, 64) != 0;
        const unsigned long long l = lane == 0 ? k.side[q] : up, s = k.k[q + 1], r = k.side[q];
        differ[q] = (lane == 0 ? k.side_ok[q] : up_ok) && k.ok[q + 1] && (unsigned)l != (unsigned)s;
        front[q] = (unsigned)(l < s ? l : s);
        differ[kAaH + q] = lane == 63 && k.side_ok[q] && (unsigned)r != (unsigned)s;
        front[kAaH + q] = (unsigned)(r < s ? r : s);
    }
#pragma unroll
    for (int q = 0; q <= kAaH; ++q) {
        const unsigned long long l = k.k[q], s = k.k[q + 1];
        differ[2 * kAaH + q] = k.ok[q] && k.ok[q + 1] && (unsigned)l != (unsigned)s;
        front[2 * kAaH + q] = (unsigned)(l < s ? l : s);
    }
#pragma unroll
    for (int q = 0; q < 3 * kAaH + 1; ++q) any = any || differ[q];
    if (__ballot(any) == 0ull) return 0;     // one triangle (most of a ground plane): no silhouette byte is needed
    unsigned char sb[3 * kAaH + 1];
#pragma unroll
    for (int q = 0; q < 3 * kAaH + 1; ++q) sb[q] = differ[q] ? sil[front[q]] : (unsigned char)0;
    bool cand = false;
#pragma unroll
    for (int q = 0; q < 3 * kAaH + 1; ++q) cand = cand || sb[q] != 0;
    if (__ballot(cand) == 0ull) return 0;
    unsigned *z = (unsigned *)g.state;
    for (int q = lane; q < kAaSlots / 4; q += 64) z[q] = 0u;
    __syncthreads();
    int n = 0;
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int q = 0; q < 3 * kAaH + 1; ++q) {
        const unsigned long long m = __ballot(sb[q] != 0);
        if (sb[q] != 0) {
            const int slot = q < kAaH ? q * kAaRow + lane
                             : q < 2 * kAaH ? (q - kAaH) * kAaRow + kAaW : kAaVert + (q - 2 * kAaH) * kAaW + lane;
            g.item[n + __popcll(m & below)] = (unsigned short)slot;
            g.state[slot] = kAaCand;
        }
        n += __popcll(m);
    }
    __syncthreads();
    return n;
}
static_assert(kAaSlots % 4 == 0, "state is cleared in words");

// Samples a and b of a slot, relative to the region's first sample.
struct AASlot {
    int ia, ja, ib, jb;
    bool horiz;
};
__device__ __forceinline__ AASlot aa_slot(int slot) {
    AASlot s;
    s.horiz = slot < kAaVert;
    if (s.horiz) {
        s.jb = slot / kAaRow;
        s.ib = slot - s.jb * kAaRow;
        s.ia = s.ib - 1;
        s.ja = s.jb;
    } else {
        s.jb = (slot - kAaVert) >> 6;
        s.ib = (slot - kAaVert) & 63;
        s.ia = s.ib;
        s.ja = s.jb - 1;
    }
    return s;
}
__device__ __forceinline__ bool aa_inside(int i, int j) { return i >= 0 && i < kAaW && j >= 0 && j < kAaH; }

// The four slots of sample (lane, row) in the order -x, +x, -y, +y, and the
// state bit that says the sample receives.
__device__ __forceinline__ int aa_slot_of(int lane, int row, int d) {
    return d < 2 ? row * kAaRow + lane + d : kAaVert + (row + d - 2) * kAaW + lane;
}
__device__ __forceinline__ constexpr unsigned char aa_self_bit(int d) { return d & 1 ? kAaA : kAaB; }

// Which sample of the pair receives: its state bit.
__device__ __forceinline__ unsigned char aa_receiver(const AAPair &pr, bool a_is_front) {
    return (pr.recv == 1) == a_is_front ? kAaB : kAaA;
}

// The candidate pairs of a workgroup's samples, compacted so that they can be
// evaluated a pair a lane.  Few samples of a wave have one, and a pair costs
// three dependent loads and some 200 instructions, many in float64: evaluated
// in place, direction by direction, every wave with a single candidate pays
// for all of its lanes four times.  Each wave lists its own pairs (sample of
// the workgroup << 2 | direction) and one barrier publishes the lists; the
// pair's result goes to the slot of that name, so a sample adds its pairs'
// terms in the order of directions whatever lane evaluated them.
template <int NT>
struct AAPairs {
    static constexpr int NW = NT / 64;
    unsigned short item[NT * 4];
    unsigned cnt[NW];
    float w[NT * 4];               // blend weight, by slot
    unsigned char state[NT * 4];   // 0: not smoothed, 1: the sample receives, 2: it gives
};

template <int NT>
__device__ __forceinline__ void aa_pairs_list(AAPairs<NT> &l, int tid, const bool (&cand)[4]) {
    const int lane = tid & 63, w = tid >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned at = 0;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const unsigned long long m = __ballot(cand[d]);
        if (cand[d]) l.item[w * 256 + at + __popcll(m & below)] = (unsigned short)(tid << 2 | d);
        at += (unsigned)__popcll(m);
    }
    if (lane == 0) l.cnt[w] = at;
}

template <int NT>
__device__ __forceinline__ unsigned aa_pairs_total(const AAPairs<NT> &l) {
    unsigned n = 0;
#pragma unroll
    for (int w = 0; w < AAPairs<NT>::NW; ++w) n += l.cnt[w];
    return n;
}

// Slot (sample << 2 | direction) of the e-th listed pair.
template <int NT>
__device__ __forceinline__ unsigned aa_pairs_item(const AAPairs<NT> &l, unsigned e) {
    unsigned base = 0;
#pragma unroll
    for (int w = 0; w < AAPairs<NT>::NW - 1; ++w)
        if (e >= l.cnt[w] && base == (unsigned)w * 256u) {
            e -= l.cnt[w];
            base += 256u;
        }
    return l.item[base + e];
}

// Renders of one camera share its keys, so the lookup, the camera smoothing and
// its adjoint do what depends on the keys alone once for a chunk of the
// camera's renders.  The chunk is the whole list unless that leaves the GPU
// under kFillBlocks workgroups, where a single camera with many renders would
// be a serial loop on an idle chip.
constexpr int kFillBlocks = 2048;
inline int render_chunk(int max_renders, long long blocks) {
    int chunk = max_renders;
    while (chunk > 1 && blocks * ((max_renders + chunk - 1) / chunk) < kFillBlocks) chunk = (chunk + 1) / 2;
    return chunk;
}

}  // namespace dsm
