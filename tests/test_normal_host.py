"""The normal numbers of the network's initial weights are those of
std::normal_distribution (GNU library), to the bit and in the same order."""
import lanes_util

SRC = """
#include <cstring>
#include "learned.h"
extern "C" long differing(int seeds, int n) {
  long bad = 0;
  for (int s = 0; s < seeds; ++s) {
    std::mt19937_64 a(s), b(s);
    std::normal_distribution<double> nd(0.0, 1.0);
    rsgdf::Normal mine;
    for (int i = 0; i < n; ++i) {
      const double x = nd(a), y = mine(b);
      bad += std::memcmp(&x, &y, sizeof x) != 0;
    }
  }
  return bad;
}
"""


def test_normal_numbers(tmp_path):
    assert lanes_util.build(tmp_path, SRC).differing(50, 5185) == 0
