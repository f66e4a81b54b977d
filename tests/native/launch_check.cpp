// Launchers of the grouped passes asked for a shape that has no kernel return
// an error and launch nothing (no device needed).
#include "ffth_launch.h"

#include <cstdio>

using namespace ffth;

template <typename T> static int check(const char* tag) {
  int bad = 0;
  GroupShape g;
  g.on = true;
  g.kcs = 1;
  g.xblocks = g.zblocks = 1;
  const int r2s[] = {1, 3, 5, 7, 12, 32};
  for (int r2 : r2s) {
    g.r2 = r2;
    if (GLaunch<T>::gz(16, g, false, 1, nullptr, nullptr, 0, 16 * r2, 1.0, -1, 0, 0) != hipErrorInvalidValue) {
      std::printf("%s: gz r2 %d\n", tag, r2);
      ++bad;
    }
  }
  g.r2 = 16;   // a tile of 256 x 16 fits no LDS
  if (GLaunch<T>::gz(256, g, false, 1, nullptr, nullptr, 0, 256, 1.0, -1, 0, 0) != hipErrorInvalidValue) {
    std::printf("%s: gz 256 x 16\n", tag);
    ++bad;
  }
  g.r2 = 4;
  if (GLaunch<T>::gz(10, g, false, 1, nullptr, nullptr, 0, 16, 1.0, -1, 0, 0) != hipErrorInvalidValue) {
    std::printf("%s: gz n0 10\n", tag);
    ++bad;
  }
  g.r1 = 5;
  if (GLaunch<T>::xinv(16, g, true, 1, nullptr, nullptr, 0, 16, 256) != hipErrorInvalidValue) {
    std::printf("%s: xinv r1 5\n", tag);
    ++bad;
  }
  return bad;
}

int main() {
  if (check<float>("float") + check<double>("double")) return 1;
  std::printf("OK\n");
  return 0;
}
