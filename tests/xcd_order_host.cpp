// The grids' orders (csrc/xcd_order.h) compiled for the host, in the forms that
// the kernels take.
#include "xcd_order.h"

// out[b]: the item of workgroup b of a gx x gy grid.  form: 0 a range per XCD, 1
// the raster's turns, 2 the tile walks' grids, 3 the camera smoothing's, 4 the
// light moments'.
extern "C" void xcd_items(int form, int gx, int gy, int *out) {
    const int n = gx * gy;
    for (int b = 0; b < n; ++b)
        out[b] = form == 0   ? dsm::xcd_remap(b, n)
                 : form == 1 ? dsm::xcd_turns<23>(b, n)
                 : form == 2 ? dsm::xcd_item<128, 4096>(b, gx, gy)
                 : form == 3 ? dsm::xcd_item<16, 8192>(b, gx, gy)
                             : dsm::xcd_item<16, 8192, true>(b, gx, gy);
}
