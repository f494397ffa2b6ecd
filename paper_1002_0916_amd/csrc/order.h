// Where a forward's order of addition is part of its result.
#pragma once

#include <stdint.h>

namespace cgh {

// Many points for the pixels: their terms add up in phase over the hologram, so
// its values are large against a residual I - T late in a fit, and the residual
// shows how the sum itself was rounded.  Another order of addition moves the
// residual's 2-norm by up to about 3.7e-4 n / pixels (z of 0.2 to 1.5 m, the points
// off by half a pixel and 10% of the amplitude: 8.7e-4 at 150x112, n = 54603; 2.7e-5
// at 365x339, n = 10048; 1.6e-5 at most over 700 clouds about the line).  Beyond the
// line the direct forwards keep one order, that of the points, whatever the launch
// looks like; below it the faster forms split the sum as suits them.
inline bool ordered_sum(int64_t n, int32_t nx, int32_t ny) {
  return 24 * n > (int64_t)nx * ny;
}

// The same for the separable variants, whose sums are the plan's K splits, each in
// order, and then the splits in order: those are shorter, and another cut moves the
// residual by up to 1.2e-5 at this line and 1.4e-4 beyond it (136x105, n = 64690).
inline bool ordered_splits(int64_t n, int32_t nx, int32_t ny) {
  return 3 * n > (int64_t)nx * ny;
}

}  // namespace cgh
