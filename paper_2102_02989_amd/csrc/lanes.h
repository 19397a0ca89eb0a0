// lanes.h -- integer rules by which the short-range kernel and the pair transforms
// deal out their lanes, for the device and for host tests.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

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

// q values per lane of the pair transforms: the image-dependent work of a term (Gaussian factor,
// bound, pair centre, E coefficients) is the same for every q, so the lanes of
// the lighter classes take several q each and do it once for all of them (s-s
// eight, p-s four, up to l_a + l_b = 3 two; the d-d accumulators leave no
// registers for more).  Measured on the 8-atom 3x3x3 workload: s-s 4 -> 8 and
// p-s 2 -> 4 took the long-range phase from 5.39 to 5.10 s; p-s 6 or
// l_a + l_b = 2 at four were slower.
__host__ __device__ constexpr int pairft_qpl(int la, int lb) {
  return la + lb == 0 ? 8 : (la + lb == 1 ? 4 : (la + lb <= 3 ? 2 : 1));
}

constexpr int kPairFtWaves = 4;  // waves of a workgroup that share a pair's terms (sliced form)

// How a class's q are dealt out.  With at least 64 q the lanes are q, and each
// takes as many of them as leave 8 waves per SIMD (a term's q-independent work
// is done once per lane: at 2400 q per class and 45 to 78 pairs, 8 q per lane
// left 2300 waves, the longest of which the launch waited for: 1x3x2 mesh, 52 ms
// of pair transforms, 26 with this rule).  With fewer than 64 q (a Gamma or small-omega build has 6
// to 30) the lanes beyond them would idle: they share the terms instead, and so
// do four waves of a workgroup where the launch has few of them.
struct PairFtShape {
  int qp, nql, waves;  // q per lane; nql > 0: sliced form
};
inline PairFtShape pairft_shape(int64_t nx, int nq, int qpmax) {
  const int64_t nw = nx * ((nq + 63) / 64);
  if (nq < 64) {
    int nql = 1;
    while (nql < nq) nql *= 2;
    return {1, nql, nw < 2048 ? kPairFtWaves : 1};
  }
  if (nw < 2048) return {1, 64, kPairFtWaves};
  int qp = qpmax;
  while (qp > 1 && nx * ((nq + 64 * qp - 1) / (64 * qp)) < 8192) qp /= 2;
  return {qp, 0, 1};
}
// blocks of q of a launch (grid y, at most 65535)
inline int64_t pairft_blocks(const PairFtShape &s, int nq) {
  const int64_t per = s.nql ? s.nql : 64 * s.qp;
  return (nq + per - 1) / per;
}

}  // namespace rsgdf
