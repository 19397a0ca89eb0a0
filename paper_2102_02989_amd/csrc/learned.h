// learned.h -- parameter layout of the screening network (FP32, host and device).
#pragma once

#include <cmath>
#include <random>

namespace rsgdf {

constexpr int kMlpF = 16;  // input features (11 used, zero padded)
constexpr int kMlpH = 64;  // hidden width
constexpr int kMlpOffMean = 0;                        // feature means [16]
constexpr int kMlpOffIstd = kMlpOffMean + kMlpF;      // 1 / feature std [16]
constexpr int kMlpOffW1 = kMlpOffIstd + kMlpF;        // [64][16]
constexpr int kMlpOffB1 = kMlpOffW1 + kMlpH * kMlpF;  // [64]
constexpr int kMlpOffW2 = kMlpOffB1 + kMlpH;          // [64][64]
constexpr int kMlpOffB2 = kMlpOffW2 + kMlpH * kMlpH;  // [64]
constexpr int kMlpOffW3 = kMlpOffB2 + kMlpH;          // [64]
constexpr int kMlpOffB3 = kMlpOffW3 + kMlpH;          // [1]
constexpr int kMlpOffLo = kMlpOffB3 + 1;              // training range, raw features [16]
constexpr int kMlpOffHi = kMlpOffLo + kMlpF;          // [16]
constexpr int kMlpNParam = kMlpOffHi + kMlpF;         // 5377
constexpr int kMlpNTrain = kMlpOffB3 + 1 - kMlpOffW1; // trainable: W1 .. b3 (5313)

// Standard normal numbers by Marsaglia's polar method: the numbers, in their order and to
// the bit, that std::normal_distribution of the GNU library draws from the generator.
// That one takes two extended-precision logarithms per uniform number, and the 5200
// weights took 170 or 330 us with where the linker put it; 60 us here.
struct Normal {
  double saved = 0.0;
  bool have = false;
  static double uniform(std::mt19937_64 &rng) {
    const double u = (double)rng() * 0x1p-64;
    return u < 1.0 ? u : std::nextafter(1.0, 0.0);
  }
  double operator()(std::mt19937_64 &rng) {
    have = !have;
    if (!have) return saved;
    double x, y, r2;
    do {
      x = 2.0 * uniform(rng) - 1.0;
      y = 2.0 * uniform(rng) - 1.0;
      r2 = x * x + y * y;
    } while (r2 > 1.0 || r2 == 0.0);
    const double m = std::sqrt(-2.0 * std::log(r2) / r2);
    saved = x * m;
    return y * m;
  }
};

}  // namespace rsgdf
