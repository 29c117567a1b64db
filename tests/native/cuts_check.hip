// Host-side driver for the test of the jet cuts' FP32 decisions: reads pairs "|eta| eta_max" (also inf,
// nan) and prints eta_side for +-eta.
#include <cstdio>
#include <cstdlib>

#include "../../paper_1002_3446_amd/csrc/bg_kernels.hpp"

int main() {
  char a[64], b[64];
  while (std::scanf("%63s %63s", a, b) == 2) {
    const float e = std::strtof(a, nullptr), m = std::strtof(b, nullptr);
    std::printf("%d %d\n", bgk::eta_side(e, m), bgk::eta_side(-e, m));
  }
  return 0;
}
