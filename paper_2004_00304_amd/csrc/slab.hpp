// slab.hpp -- where a slab's buffers lie, in the particles' own coordinate.
// Plain C++ (no HIP types), so that the tests compile the same source.
#pragma once

#include <math.h>

namespace lbmpcd {

// The exchange redraws the particles whose fine row clamp(floor((y - ylo) r),
// 0, R - 1) lies in the lower buf_lo or the upper buf_hi node rows.  For
// binary32 positions y - ylo and its product with r are exact in binary64, so
// that rule is y < below or y >= from, with these two bounds.  The clamp
// belongs to it: a position outside the slab has the row of the face next to
// it, and y = yhi occurs (the initial positions are rounded to binary32).  A
// face without a buffer therefore has no bound (no y is below -inf, none
// compares with NaN), and where one buffer fills the slab every y is in it.
inline void buffer_bounds(int ylo, int yhi, int buf_lo, int buf_hi, float* below, float* from) {
    if (buf_lo >= yhi - ylo || buf_hi >= yhi - ylo) {
        *below = *from = -INFINITY;
        return;
    }
    *below = buf_lo > 0 ? (float)(ylo + buf_lo) : -INFINITY;
    *from = buf_hi > 0 ? (float)(yhi - buf_hi) : NAN;
}

}  // namespace lbmpcd
