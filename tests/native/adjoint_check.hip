// Host-side driver for the tests of the gradient's adjoints: reads lines "Q r1 r2 r3 r4 qb0..qb3" in
// hexadecimal and prints the four words of rambo_q_adj.
#include <cstdio>
#include <cstdlib>

#include "../../paper_1002_3446_amd/csrc/bg_adjoint.hpp"

namespace {
double word() {
  char s[64];
  if (std::scanf("%63s", s) != 1) std::exit(1);
  return std::strtod(s, nullptr);
}
}  // namespace

int main() {
  char tag[4];
  while (std::scanf("%3s", tag) == 1) {
    if (tag[0] == 'Q') {
      double r[4], qb[4], rb[4];
      for (double& x : r) x = word();
      for (double& x : qb) x = word();
      bgk::rambo_q_adj(r[0], r[1], r[2], r[3], qb, rb);
      std::printf("%a %a %a %a\n", rb[0], rb[1], rb[2], rb[3]);
    } else {
      return 1;
    }
  }
  return 0;
}
