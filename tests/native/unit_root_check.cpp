// Compile-time twiddle factors: every axis length's table within 0.51 units in
// the last place of 1 (half a unit is rounding; the fixed-point series is off
// by less than 2^-60) of the long-double cosine and sine, exact on the axes.
#include "unit_root.h"

#include <cmath>
#include <cstdio>

int main() {
  const int lens[] = {1, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 256, 512, 768, 1024};
  for (int n : lens)
    for (int m = 0; m < n; ++m) {
      double c = 2.0, s = 2.0;
      ffth::unit_root(m, n, c, s);
      // first-octant arguments in long double: cosl and sinl are exact to 2^-64 there
      const int o = 8 * m / n, rem = 8 * m - o * n;
      const long double x = 0.785398163397448309615660845819875721L * (o & 1 ? n - rem : rem) / n;
      const bool swap = (o + 1) & 2;
      long double rc = swap ? sinl(x) : cosl(x), rs = swap ? cosl(x) : sinl(x);
      if (o >= 2 && o < 6) rc = -rc;
      if (o >= 4) rs = -rs;
      const long double tol = 0.51L / 9007199254740992.0L;   // values below 1: 2^-53 between neighbours
      if (fabsl(c - rc) > tol || fabsl(s - rs) > tol) {
        std::printf("n %d m %d: %.3Le %.3Le\n", n, m, fabsl(c - rc), fabsl(s - rs));
        return 1;
      }
      if (4 * m % n == 0 && (c * c + s * s != 1.0 || c * s != 0.0)) {
        std::printf("n %d m %d: not on the axis\n", n, m);
        return 1;
      }
    }
  // one of them at compile time, as the tables are
  struct R {
    double c, s;
    constexpr R() : c(0), s(0) { ffth::unit_root(5, 96, c, s); }
  };
  constexpr R r;
  static_assert(r.c > 0.94 && r.c < 0.95 && r.s > 0.32 && r.s < 0.33, "unit_root(5, 96)");
  std::printf("OK\n");
  return 0;
}
