// Consuming kernels of the radius relation on tiles of 16 destinations (rows of up to kTileFeatFwd features forward,
// kTileFeatBwd backward).
#pragma once

#include "radius_cells.hpp"

namespace tiga {
namespace radius {

constexpr int kTileFeatFwd = 64;
constexpr int kTileFeatBwd = 32;

// Whether rows of `feat` floats of n points have 32-bit byte offsets.
inline bool tile_offsets(int64_t n, int64_t feat) { return n * feat * 4 < (int64_t{1} << 32); }

// y (and count) of feat <= kTileFeatFwd; `cells` the sorted cell ids (one per record).
int tile_forward(int64_t n, int32_t feat, const Cells &c, const int32_t *cells, const float *x, float r2, float nis,
                 float *y, int32_t *count, hipStream_t stream);

// dx and dpos (either may be null) of feat <= kTileFeatBwd.
int tile_backward(int64_t n, int32_t feat, const Cells &c, const int32_t *cells, const float *x, const float *dy,
                  float r2, float nis, float tis, float *dx, float *dpos, hipStream_t stream);

}  // namespace radius
}  // namespace tiga
