// lanes.h -- integer rules by which the short-range kernel deals out its lanes,
// for the device and for host tests.
#pragma once
#include <hip/hip_runtime.h>

namespace rsgdf {

// Work of a pair image kept up to R_c window wm (0 .. 255): the sphere its lattice
// vectors lie in, in cubes of the window width.  A whole number, so that sums over
// the 64 images of a batch are exact and grow with every image (2^30 at most).
__host__ __device__ inline int sr_image_weight(int wm) { return (wm + 1) * (wm + 1) * (wm + 1); }

// Image j of a batch of m owns rows [sr_row_end(j - 1), sr_row_end(j)) of `rows` >= m:
// one at least, the others in proportion to its weight.  cum: weight of the images
// up to j; inv_tot: 1 / weight of all.  cum increases with j and every step below
// keeps that order, so no image is left without a row, however the floats round.
__host__ __device__ inline int sr_row_end(int j, int m, int rows, int cum, float inv_tot) {
  return j == m - 1 ? rows : j + 1 + (int)((float)(rows - m) * ((float)cum * inv_tot));
}

}  // namespace rsgdf
