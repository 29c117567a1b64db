// Host-side driver for the tests of the gradient's adjoints: reads lines in hexadecimal and prints the
// results of "Q r1 r2 r3 r4 qb0..qb3" (rambo_q_adj), "P px py pz h er1 er2 er3 ei1 ei2" (polarisation_adj,
// h = +-1) and "I Q0..Q3 sqrt(s) bxb byb bzb gammab ab Xb" (rambo_init_adj after RamboMap::init).
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
      bgk::rambo_q_adj(r[0], r[1], r[2], r[3], -bgk::log_fp64(r[2] * r[3]), qb, rb);
      std::printf("%a %a %a %a\n", rb[0], rb[1], rb[2], rb[3]);
    } else if (tag[0] == 'P') {
      double p[4] = {0.0}, er[4] = {0.0}, ei[4] = {0.0}, pb[4] = {0.0};
      for (int mu = 1; mu < 4; ++mu) p[mu] = word();
      const bool plus = word() > 0.0;
      for (int mu = 1; mu < 4; ++mu) er[mu] = word();
      for (int mu = 1; mu < 3; ++mu) ei[mu] = word();
      bgk::polarisation_adj(p, plus, er, ei, pb);
      std::printf("%a %a %a\n", pb[1], pb[2], pb[3]);
    } else if (tag[0] == 'I') {
      double Q[4], Qb[4] = {0.0}, sb = 0.0;
      for (double& x : Q) x = word();
      bgk::RamboMap m;
      m.init(Q, word());
      bgk::RamboMapAdj A;
      for (double* x : {&A.bxb, &A.byb, &A.bzb, &A.gammab, &A.ab, &A.Xb}) *x = word();
      bgk::rambo_init_adj(m, Q, A, Qb, sb);
      std::printf("%a %a %a %a %a\n", Qb[0], Qb[1], Qb[2], Qb[3], sb);
    } else {
      return 1;
    }
  }
  return 0;
}
