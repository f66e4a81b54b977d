// Twiddle factors at compile time (no HIP: also compiled by the host tests).
#pragma once
#include <stdint.h>

namespace ffth {

// cos and sin of 2 pi m / n, 0 <= m < n: Taylor series in the first octant, in
// fixed point with 62 fractional bits (error below 2^-60), rounded to FP64
// once.  The same series in FP64 rounds at every step and came out up to 1.26e-16
// off (correctly rounded values: 5.6e-17), which the transforms pass on: each
// output carries the error of as many factors as it has stages.
constexpr void unit_root(int m, int n, double& c, double& s) {
  typedef __int128 i128;
  const int64_t one = INT64_C(1) << 62, pi4 = INT64_C(3622009729038561421);   // 1 and pi / 4
  // angle = (pi / 4) (o + r), r in [0, 1): odd octants are measured from their end
  const int o = 8 * m / n, rem = 8 * m - o * n;
  const int64_t x = (int64_t)(((i128)pi4 * (o & 1 ? n - rem : rem) + n / 2) / n), x2 = (int64_t)(((i128)x * x) >> 62);
  int64_t a = one, b = one;   // cos x and sin x / x
  for (int k = 20; k >= 2; k -= 2) {
    a = one - (int64_t)(((i128)a * x2) >> 62) / (k * (k - 1));
    b = one - (int64_t)(((i128)b * x2) >> 62) / (k * (k + 1));
  }
  b = (int64_t)(((i128)b * x) >> 62);
  const bool swap = (o + 1) & 2;   // octants 1, 2, 5, 6
  const double unit = 1.0 / (double)one;
  c = (double)(swap ? b : a) * unit;
  s = (double)(swap ? a : b) * unit;
  if (o >= 2 && o < 6) c = -c;
  if (o >= 4) s = -s;
}

}  // namespace ffth
