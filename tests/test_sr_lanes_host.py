"""Host tests of the rules by which the short-range kernel and the pair transforms deal
out their lanes (csrc/lanes.h), compiled for the CPU."""
import ctypes

import numpy as np
import pytest

import lanes_util

SRC = """
#include "lanes.h"
extern "C" void row_ends(const int *wm, int m, int rows, int *out) {
  int tot = 0, cum = 0;
  for (int j = 0; j < m; ++j) tot += rsgdf::sr_image_weight(wm[j]);
  const float inv = 1.0f / (float)tot;
  for (int j = 0; j < m; ++j) {
    cum += rsgdf::sr_image_weight(wm[j]);
    out[j] = rsgdf::sr_row_end(j, m, rows, cum, inv);
  }
}
extern "C" long box_errors(int dim0, int dim1, int dim2, int near) {
  const int d12 = dim1 * dim2, nbox = dim0 * d12;
  const float inv12 = 1.0f / (float)d12, inv2 = 1.0f / (float)dim2;
  long bad = 0;
  for (int j0 = 0; j0 < dim0; ++j0)
    for (int k = -near; k <= near; ++k) {
      const int q = j0 * d12 + k;
      if (q < 0 || q >= nbox) continue;
      int a, b, c;
      rsgdf::sr_box_entry(q, dim1, dim2, inv12, inv2, a, b, c);
      bad += a != q / d12 || b != q / dim2 % dim1 || c != q % dim2;
    }
  return bad;
}
extern "C" long pairft_blocks(long nx, int nq, int la, int lb) {
  return rsgdf::pairft_blocks(rsgdf::pairft_shape(nx, nq, rsgdf::pairft_qpl(la, lb)), nq);
}
"""


@pytest.fixture(scope="module")
def lanes(tmp_path_factory):
    return lanes_util.build(tmp_path_factory.mktemp("lanes"), SRC)


def _row_ends(lanes, wm, rows):
    wm = np.ascontiguousarray(wm, np.int32)
    out = np.zeros(len(wm), np.int32)
    p = ctypes.POINTER(ctypes.c_int)
    lanes.row_ends(wm.ctypes.data_as(p), len(wm), rows, out.ctypes.data_as(p))
    return out


def test_every_image_gets_a_row(lanes):
    """Near images with hundreds of windows beside far ones with a few: the running
    sum of volumes in single precision is not monotone there (64 values, summed in the
    order of a wave's scan), and images were left without a row."""
    rng = np.random.default_rng(0)
    decreasing = 0
    for _ in range(4000):
        rows = int(rng.integers(2, 65))
        m = int(rng.integers(1, rows + 1))
        far = rng.random(m) < rng.choice([0.1, 0.5, 0.9])
        wm = np.where(far, rng.integers(0, 6, m), rng.integers(75, 256, m))
        e = _row_ends(lanes, wm, rows)
        assert e[-1] == rows and e[0] >= 1 and np.all(np.diff(e) >= 1), (rows, wm.tolist(), e.tolist())
        f = (np.float32(wm + 1) ** 3 * np.float32(10.0 ** rng.uniform(-8, 0))).astype(np.float32)
        o = 1
        while o < m:
            f[o:] = f[o:] + f[:-o].copy()
            o *= 2
        decreasing += bool(np.any(np.diff(f) < 0))
    assert decreasing > 100  # the inputs are of the kind that matters
    for rows in (1, 7, 64):  # the extremes
        for wm in ([255] * rows, [0] * rows, [255] + [0] * (rows - 1), [0] * (rows - 1) + [255]):
            e = _row_ends(lanes, wm, rows)
            assert e.tolist() == list(range(1, rows + 1))


def test_rows_follow_the_weights(lanes):
    """One image of weight 27 against one of 1 over 64 rows: 62 rows are shared 27 to 1."""
    assert _row_ends(lanes, [2, 0], 64).tolist() == [1 + 62 * 27 // 28, 64]


@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 5, 7), (1, 1, 1000), (1000, 1, 1), (161, 161, 161), (172, 173, 171),
                                  (257, 256, 255), (400, 401, 399), (1000, 999, 1001), (1001, 1000, 1000)])
def test_box_entries(lanes, dims):
    """Boxes of lattice vectors up to the size the planner accepts (|M| < 500): every
    entry near a plane's end has the indices of the whole-number division."""
    lanes.box_errors.restype = ctypes.c_long
    assert lanes.box_errors(*dims, min(4 * dims[2] + 200, dims[1] * dims[2])) == 0


@pytest.mark.parametrize("la,lb,width", [(0, 0, 8), (1, 0, 4), (1, 1, 2), (2, 1, 2), (2, 2, 1)])
def test_pair_transform_grid(lanes, la, lb, width):
    """A class of up to 65535 blocks of 64 width q is one launch, down to one pair."""
    lanes.pairft_blocks.restype = ctypes.c_long
    for nx in (1, 21, 10000):
        assert lanes.pairft_blocks(ctypes.c_long(nx), 65535 * 64 * width, la, lb) == 65535
        assert lanes.pairft_blocks(ctypes.c_long(nx), 65535 * 64 * width + 1, la, lb) == 65536
