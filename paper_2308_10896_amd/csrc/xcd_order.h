// The order in which a grid's workgroups take their items on the 8 XCDs.  The
// functions run on the host too, where they are tested.
#pragma once

#include <hip/hip_runtime.h>

namespace dsm {

// Workgroups are dispatched to the 8 XCDs round-robin by linear id, and each
// XCD has its own L2.  These renumber a grid so that each XCD takes a
// contiguous range of work items: neighbouring tiles and rows, which share
// cache lines and halos, then share an L2.  Both are bijections, so any
// dispatch order stays correct.
__host__ __device__ __forceinline__ int xcd_remap(int b, int n) {
    constexpr int kXcd = 8;
    const int xcd = b % kXcd, idx = b / kXcd;
    const int per = n / kXcd, rem = n % kXcd;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

// The same with the XCDs taking turns of `run` consecutive items, which evens
// out ranges that cost more than others; the last items, too few for a turn, are
// split as above.
template <int RUN>
__host__ __device__ __forceinline__ int xcd_turns(int b, int n) {
    constexpr int kTurn = 8 * RUN;
    const int whole = n / kTurn * kTurn;
    return b < whole ? b / kTurn * kTurn + b % 8 * RUN + b / 8 % RUN : whole + xcd_remap(b - whole, n - whole);
}

// Item of workgroup b in a grid of gx items in each of gy views.  Where every XCD gets whole views (or nearly, of
// 32 and more) a contiguous range is even, and a view's maps stay in one L2;
// otherwise one XCD's range is sky and another's the object, and they take
// turns: a 1080p camera's lookup adjoint 110 -> 81 us, three 2048^2 maps' light
// adjoint 174 -> 153 (turns with 64 views instead: 388 -> 434 and 187 -> 188).
// SPREAD: turns with many views too, for kernels that read little but their own
// region.  Grids under FROM workgroups keep the ranges (a cube light's six small
// maps 170 us a pass, 172 in turns); of 4,096 tiles on, turns pay (a 512^2 view's
// lookup adjoint 19 -> 13 us).
template <int RUN, int FROM, bool SPREAD = false>
__host__ __device__ __forceinline__ int xcd_item(int b, int gx, int gy) {
    const int n = gx * gy;
    const bool range = n < FROM || (!SPREAD && (gy % 8 == 0 || gy >= 32));
    return range ? xcd_remap(b, n) : xcd_turns<RUN>(b, n);
}

}  // namespace dsm
