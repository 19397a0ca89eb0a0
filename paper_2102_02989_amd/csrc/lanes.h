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

// Entry q of a box of dim1 x dim2 planes (j0, j1, j2 in row order), the divisions
// by reciprocals: inv12 = 1 / (dim1 dim2), inv2 = 1 / dim2.  Up to 2^30 entries and
// 1024 along an axis the quotient in single precision is off by one at most next to
// a plane's end (from 4e6 entries on), which the remainder shows; j1 is exact.
__host__ __device__ inline void sr_box_entry(int q, int dim1, int dim2, float inv12, float inv2, int &j0, int &j1,
                                             int &j2) {
  const int d12 = dim1 * dim2;
  j0 = (int)(((float)q + 0.5f) * inv12);
  int r0 = q - j0 * d12;
  const int fix = (r0 >= d12) - (r0 < 0);
  j0 += fix;
  r0 -= fix * d12;
  j1 = (int)(((float)r0 + 0.5f) * inv2);
  j2 = r0 - j1 * dim2;
}

}  // namespace rsgdf
