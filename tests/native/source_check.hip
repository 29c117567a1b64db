// Host-side driver for the test of the FP64 helicity sources: prints, in hexadecimal, momenta spread
// over 20 decades of scale, some along the beam axis, and the words of polarisation<double> for
// both helicities.
#include <cstdint>
#include <cstdio>

#include "../../paper_1002_3446_amd/csrc/bg_device.hpp"

int main() {
  uint64_t st = 0x9E3779B97F4A7C15ull;
  auto next = [&]() {
    st ^= st << 13;
    st ^= st >> 7;
    st ^= st << 17;
    return st;
  };
  for (int i = 0; i < 100000; ++i) {
    const double scale = std::pow(10.0, (double)(int)(next() % 21) - 10.0);
    double p[4] = {0.0, 0.0, 0.0, 0.0};
    for (int mu = 1; mu < 4; ++mu) p[mu] = scale * ((double)(int64_t)next() * 0x1p-63);
    if (i % 250 == 0) p[1] = p[2] = 0.0;
    const bool plus = i & 1;
    const bgk::cv4<double> e = bgk::polarisation<double>(p, plus);
    std::printf("%d %a %a %a", (int)plus, p[1], p[2], p[3]);
    for (int mu = 0; mu < 4; ++mu) std::printf(" %a %a", e.re[mu], e.im[mu]);
    std::printf("\n");
  }
  return 0;
}
