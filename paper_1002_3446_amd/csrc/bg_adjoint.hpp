// Hand-written adjoint of the event path: d log w_int / d(RAMBO uniforms, x1, x2).
//
// log w_int = a log x1 + b log(1-x1) + a log x2 + b log(1-x2) + (n-5) log s_hat + log|A|^2 + c
// (the integrand of Eq. 3.8 without the cut step function and without the sampling density;
// the flux 1/s_hat and RAMBO's volume s_hat^(n-4) give the s_hat power).  |A|^2 is evaluated on
// the partonic centre-of-mass momenta, so the reverse sweep runs: closure -> recursion
// (Eqs. 3.1-3.2, regrouped as in the forward) -> helicity sources -> momenta -> RAMBO's
// conformal map -> q(rho) -> uniforms, and sqrt(s_hat) -> x1, x2.  The forward is recomputed
// in the kernel; no current is kept between the two calls of the torch Function.
//
// Complex adjoints are carried as zb = dL/dRe z + i dL/dIm z, so for a bilinear w = x y the
// rule is xb += conj(y) wb, and a real factor r of a complex z gets rb += Re(conj(z) wb).
#pragma once

#include "bg_group_adj.hpp"
#include "bg_kernels.hpp"
#include "bg_launch.hpp"

namespace bgk {

template <typename T>
__device__ __forceinline__ T gsign(int mu) {
  return mu == 0 ? T(1) : T(-1);
}

// r + i i = x . k for a contravariant real four-vector k (the reverse sweep keeps its span
// momenta contravariant)
template <typename T>
__device__ __forceinline__ void rdot_contra(const cv4<T>& x, const T k[4], T& r, T& i) {
  r = x.re[0] * k[0];
  i = x.im[0] * k[0];
#pragma unroll
  for (int mu = 1; mu < 4; ++mu) {
    r = fmac(-x.re[mu], k[mu], r);
    i = fmac(-x.im[mu], k[mu], i);
  }
}

// from d = x.y (bilinear Minkowski): xb_mu += g_mu conj(y_mu) db
template <typename T>
__device__ __forceinline__ void cdot_adj(const cv4<T>& y, T dbr, T dbi, cv4<T>& xb) {
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    const T g = gsign<T>(mu);
    xb.re[mu] = fmac(g * y.im[mu], dbi, fmac(g * y.re[mu], dbr, xb.re[mu]));
    xb.im[mu] = fmac(-g * y.im[mu], dbr, fmac(g * y.re[mu], dbi, xb.im[mu]));
  }
}

// from acc += c y (complex c): yb += conj(c) accb
template <typename T>
__device__ __forceinline__ void caxpy_adj_y(T cr, T ci, const cv4<T>& accb, cv4<T>& yb) {
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    yb.re[mu] = fmac(ci, accb.im[mu], fmac(cr, accb.re[mu], yb.re[mu]));
    yb.im[mu] = fmac(-ci, accb.re[mu], fmac(cr, accb.im[mu], yb.im[mu]));
  }
}

// from acc += c y: cb += sum_mu conj(y_mu) accb_mu
template <typename T>
__device__ __forceinline__ void caxpy_adj_c(const cv4<T>& y, const cv4<T>& accb, T& cbr, T& cbi) {
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    cbr = fmac(y.im[mu], accb.im[mu], fmac(y.re[mu], accb.re[mu], cbr));
    cbi = fmac(-y.im[mu], accb.re[mu], fmac(y.re[mu], accb.im[mu], cbi));
  }
}

// add a span-momentum adjoint to each of the legs A..B
template <int A, int B, int L, typename T>
__device__ __forceinline__ void spread(const T Kb[4], T (&kb)[L][4]) {
  static_for<A, B + 1>([&](auto tc) {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) kb[decltype(tc)::value][mu] += Kb[mu];
  });
}

// Reverse of span_vertex for span [A..B]: given Vb (adjoint of its bracket sum V) and the
// adjoint (sbr, sbi) of its scalar S, accumulate into the adjoints of the sub-currents,
// sub-span scalars and leg momenta.
template <int L, int A, int B, typename T>
__device__ __forceinline__ void span_vertex_adj(const double (&k)[L][4], const cv4<T> (&J)[Spans<L>::count],
                                                const T (&Sr)[Spans<L>::count], const T (&Si)[Spans<L>::count],
                                                const cv4<T>& Vb, T sbr, T sbi, cv4<T> (&Jb)[Spans<L>::count],
                                                T (&Sbr)[Spans<L>::count], T (&Sbi)[Spans<L>::count],
                                                T (&kb)[L][4]) {
  using SP = Spans<L>;
  // V = 2X + Y
  cv4<T> Xb, Yb;
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    Xb.re[mu] = T(2) * Vb.re[mu];
    Xb.im[mu] = T(2) * Vb.im[mu];
    Yb.re[mu] = Vb.re[mu];
    Yb.im[mu] = Vb.im[mu];
  }
  // Y -= S[A..j] J[j+1..B]  and  Y -= S[i+1..B] J[A..i]
  static_for<A + 1, B>([&](auto jc) {
    constexpr int j = decltype(jc)::value, Sx = SP::at(A, j), Jx = SP::at(j + 1, B);
    T cr = T(0), ci = T(0);
    caxpy_adj_c(J[Jx], Yb, cr, ci);
    Sbr[Sx] -= cr;
    Sbi[Sx] -= ci;
    caxpy_adj_y(-Sr[Sx], -Si[Sx], Yb, Jb[Jx]);
  });
  static_for<A, B - 1>([&](auto ic) {
    constexpr int i = decltype(ic)::value, Sx = SP::at(i + 1, B), Jx = SP::at(A, i);
    T cr = T(0), ci = T(0);
    caxpy_adj_c(J[Jx], Yb, cr, ci);
    Sbr[Sx] -= cr;
    Sbi[Sx] -= ci;
    caxpy_adj_y(-Sr[Sx], -Si[Sx], Yb, Jb[Jx]);
  });
  // X += (J[A..i] . J[j+1..B]) J[i+1..j]
  static_for<A, B - 1>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    static_for<i + 1, B>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      constexpr int PA = SP::at(A, i), PM = SP::at(i + 1, j), PC = SP::at(j + 1, B);
      T er, ei;
      cdot(J[PA], J[PC], er, ei);
      T ebr = T(0), ebi = T(0);
      caxpy_adj_c(J[PM], Xb, ebr, ebi);
      caxpy_adj_y(er, ei, Xb, Jb[PM]);
      cdot_adj(J[PC], ebr, ebi, Jb[PA]);
      cdot_adj(J[PA], ebr, ebi, Jb[PC]);
    });
  });
  // three-gluon brackets
  static_for<A, B>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr int PA = SP::at(A, i), PB = SP::at(i + 1, B);
    double KAd[4], KBd[4];
    span_sum<A, i, L>(k, KAd);
    span_sum<i + 1, B, L>(k, KBd);
    T ka[4], kbv[4];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      ka[mu] = T(KAd[mu]);
      kbv[mu] = T(KBd[mu]);
    }
    T dr, di, ar, ai, br, bi;
    cdot(J[PA], J[PB], dr, di);
    rdot_contra(J[PA], kbv, ar, ai);
    rdot_contra(J[PB], ka, br, bi);
    // X += ca J[PB] - cb J[PA]
    T cabr = T(0), cabi = T(0), cbbr = T(0), cbbi = T(0);
    caxpy_adj_c(J[PB], Xb, cabr, cabi);
    caxpy_adj_y(ar, ai, Xb, Jb[PB]);
    caxpy_adj_c(J[PA], Xb, cbbr, cbbi);
    cbbr = -cbbr;
    cbbi = -cbbi;
    caxpy_adj_y(-br, -bi, Xb, Jb[PA]);
    // Y += d (KA - KB);  S += d
    T dbr = sbr, dbi = sbi;
    T KAb[4], KBb[4];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      const T dk = ka[mu] - kbv[mu];
      dbr += dk * Yb.re[mu];
      dbi += dk * Yb.im[mu];
      const T w = dr * Yb.re[mu] + di * Yb.im[mu];  // Re(conj(d) Yb_mu)
      KAb[mu] = w;
      KBb[mu] = -w;
    }
    // d = J[PA] . J[PB]
    cdot_adj(J[PB], dbr, dbi, Jb[PA]);
    cdot_adj(J[PA], dbr, dbi, Jb[PB]);
    // ca = J[PA] . KB,  cb = J[PB] . KA
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      const T g = gsign<T>(mu);
      Jb[PA].re[mu] += g * kbv[mu] * cabr;
      Jb[PA].im[mu] += g * kbv[mu] * cabi;
      KBb[mu] += g * (J[PA].re[mu] * cabr + J[PA].im[mu] * cabi);
      Jb[PB].re[mu] += g * ka[mu] * cbbr;
      Jb[PB].im[mu] += g * ka[mu] * cbbi;
      KAb[mu] += g * (J[PB].re[mu] * cbbr + J[PB].im[mu] * cbbi);
    }
    spread<A, i, L, T>(KAb, kb);
    spread<i + 1, B, L, T>(KBb, kb);
  });
}

// Reverse sweep of bg_forward + closure.  mb: adjoint of m = eps0 . V.  Outputs the adjoints
// of the sources (srcb), of the closing polarisation (e0b) and of the scaled leg momenta (kb).
template <int L, typename T>
__device__ __forceinline__ void bg_reverse(const double (&k)[L][4], const cv4<T> (&J)[Spans<L>::count],
                                           const T (&Sr)[Spans<L>::count], const T (&Si)[Spans<L>::count],
                                           const cv4<T>& eps0, const cv4<T>& Vfull, T mbr, T mbi,
                                           cv4<T> (&srcb)[L], cv4<T>& e0b, T (&kb)[L][4]) {
  using SP = Spans<L>;
  cv4<T> Jb[SP::count];
  T Sbr[SP::count], Sbi[SP::count];
  static_for<0, SP::count>([&](auto sc) {
    constexpr int s = decltype(sc)::value;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) Jb[s].re[mu] = Jb[s].im[mu] = T(0);
    Sbr[s] = Sbi[s] = T(0);
  });
  static_for<0, L>([&](auto tc) {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) kb[decltype(tc)::value][mu] = T(0);
  });
  // m = eps0 . V
  cv4<T> Vb;
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) Vb.re[mu] = Vb.im[mu] = e0b.re[mu] = e0b.im[mu] = T(0);
  cdot_adj(eps0, mbr, mbi, Vb);
  cdot_adj(Vfull, mbr, mbi, e0b);
  span_vertex_adj<L, 0, L - 1, T>(k, J, Sr, Si, Vb, T(0), T(0), Jb, Sbr, Sbi, kb);
  // lengths L-1 down to 2
  static_for<0, L - 2>([&](auto rc) {
    constexpr int len = L - 1 - decltype(rc)::value;
    static_for<0, L - len + 1>([&](auto ac) {
      constexpr int a = decltype(ac)::value, b = a + len - 1, s = SP::at(a, b);
      double Kd[4];
      span_sum<a, b, L>(k, Kd);
      const T prop = T(1.0 / minkowski_sq(Kd));
      // J = V prop:  Vb = prop Jb;  K_mu gets -2 g_mu K_mu prop sum Re(conj(J) Jb)
      cv4<T> Vbs;
      T rj = T(0);
#pragma unroll
      for (int mu = 0; mu < 4; ++mu) {
        Vbs.re[mu] = prop * Jb[s].re[mu];
        Vbs.im[mu] = prop * Jb[s].im[mu];
        rj += J[s].re[mu] * Jb[s].re[mu] + J[s].im[mu] * Jb[s].im[mu];
      }
      T Kb[4];
#pragma unroll
      for (int mu = 0; mu < 4; ++mu) Kb[mu] = T(-2) * gsign<T>(mu) * T(Kd[mu]) * prop * rj;
      spread<a, b, L, T>(Kb, kb);
      span_vertex_adj<L, a, b, T>(k, J, Sr, Si, Vbs, Sbr[s], Sbi[s], Jb, Sbr, Sbi, kb);
    });
  });
  static_for<0, L>([&](auto tc) { srcb[decltype(tc)::value] = Jb[decltype(tc)::value]; });
}

// Adjoint of polarisation(): accumulates dL/dp (spatial components) from the adjoints of the
// source's words that are not identically zero (re[1..3], im[1], im[2]).  Every coefficient is one
// rounded quotient of products (the quotients by one number share its reciprocal): along and across the
// polar angle with reciprocal roots, the result was 1.5 times further from its exact value.
__host__ __device__ __forceinline__ void polarisation_adj(const double p[4], bool plus, const double (&er)[4],
                                                          const double (&ei)[4], double pb[4]) {
  const double px = p[1], py = p[2], pz = p[3];
  const double pt2 = px * px + py * py;
  if (!(pt2 > 0.0)) return;  // a leg along the beam axis: its direction is fixed
  const double pa = sqrt_fp64(pt2 + pz * pz), pt = sqrt_fp64(pt2), ipt = recip_refine(pt);
  const double ct = div_fp64(pz, pa), cf = div_refined(px, pt, ipt), sf = div_refined(py, pt, ipt);
  const double r = 0.70710678118654752440;
  const double hs = plus ? 1.0 : -1.0;
  const double ctb = -hs * r * (cf * er[1] + sf * er[2]);
  const double stb = hs * r * er[3];
  const double cfb = -hs * r * ct * er[1] - r * ei[2];
  const double sfb = r * ei[1] - hs * r * ct * er[2];
  const double a3 = pa * pa * pa, t3 = pt2 * pt, m3 = pt * a3;
  const double ia3 = recip_refine(a3), it3 = recip_refine(t3), im3 = recip_refine(m3);
  pb[1] += ctb * div_refined(-pz * px, a3, ia3) + stb * div_refined(px * pz * pz, m3, im3) +
           cfb * div_refined(py * py, t3, it3) + sfb * div_refined(-px * py, t3, it3);
  pb[2] += ctb * div_refined(-pz * py, a3, ia3) + stb * div_refined(py * pz * pz, m3, im3) +
           cfb * div_refined(-px * py, t3, it3) + sfb * div_refined(px * px, t3, it3);
  pb[3] += ctb * div_refined(pt2, a3, ia3) + stb * div_refined(-pt * pz, a3, ia3);
}

struct RamboMapAdj {
  double bxb, byb, bzb, gammab, ab, Xb;
};

// Adjoint of RamboMap::apply for one particle.
__device__ __forceinline__ void rambo_apply_adj(const RamboMap& m, const double q[4], const double pb[4], double qb[4],
                                                RamboMapAdj& A) {
  const double b[3] = {m.bx, m.by, m.bz};
  const double bq = b[0] * q[1] + b[1] * q[2] + b[2] * q[3];
  double inner = m.gamma * q[0] + bq;
  A.Xb += pb[0] * inner;
  const double e = m.X * pb[0];
  A.gammab += e * q[0];
  qb[0] += e * m.gamma;
  double bqb = e;
  double bb[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    inner = q[j + 1] + b[j] * q[0] + m.a * bq * b[j];
    A.Xb += pb[j + 1] * inner;
    const double P = m.X * pb[j + 1];
    qb[j + 1] += P;
    bb[j] += P * q[0] + P * m.a * bq;
    qb[0] += P * b[j];
    A.ab += P * bq * b[j];
    bqb += P * m.a * b[j];
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    bb[j] += bqb * q[j + 1];
    qb[j + 1] += bqb * b[j];
  }
  A.bxb += bb[0];
  A.byb += bb[1];
  A.bzb += bb[2];
}

// Adjoint of RamboMap::init: accumulates dL/dQ and dL/dsqrt(s_hat); every quotient by M rounded.
__host__ __device__ __forceinline__ void rambo_init_adj(const RamboMap& m, const double Q[4], const RamboMapAdj& A,
                                                        double Qb[4], double& sb) {
  const double M = sqrt_fp64(Q[0] * Q[0] - Q[1] * Q[1] - Q[2] * Q[2] - Q[3] * Q[3]), iM = recip_refine(M);
  sb += div_refined(A.Xb, M, iM);
  double Mb = div_refined(-A.Xb * m.X, M, iM);
  const double gammab = A.gammab - A.ab * m.a * m.a;
  Qb[0] += div_refined(gammab, M, iM);
  Mb += div_refined(-gammab * m.gamma, M, iM);
  const double b[3] = {m.bx, m.by, m.bz};
  const double bb[3] = {A.bxb, A.byb, A.bzb};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    Qb[j + 1] += div_refined(-bb[j], M, iM);
    Mb += div_refined(-bb[j] * b[j], M, iM);
  }
  const double M2b = div_refined(0.5 * Mb, M, iM);
  Qb[0] += 2.0 * Q[0] * M2b;
#pragma unroll
  for (int j = 0; j < 3; ++j) Qb[j + 1] += -2.0 * Q[j + 1] * M2b;
}

// Adjoint of rambo_q: rho adjoints from q adjoints, with no division by q0 (zero where r3 r4 = 1);
// at r1 = 0 or 1 the derivative in r1 is infinite and the others are finite.  q0: the energy,
// -log_fp64(r3 r4), from rambo_q.
__host__ __device__ __forceinline__ void rambo_q_adj(double r1, double r2, double r3, double r4, double q0,
                                                     const double qb[4], double rb[4]) {
  const double c = 2.0 * r1 - 1.0;
  const double st = sqrt_fp64(1.0 - c * c);
  double sp, cp;
  sincospi_fp64(2.0 * r2, &sp, &cp);
  const double q0b = qb[0] + qb[1] * st * cp + qb[2] * st * sp + qb[3] * c;
  const double stb = q0 * (qb[1] * cp + qb[2] * sp);
  const double cpb = q0 * st * qb[1], spb = q0 * st * qb[2];
  const double cb = q0 * qb[3] - stb * c / st;
  rb[0] = 2.0 * cb;
  rb[1] = 2.0 * 3.14159265358979323846 * (cp * spb - sp * cpb);
  rb[2] = -q0b / r3;
  rb[3] = -q0b / r4;
}

// Per-event kinematics of the gradient kernels (partonic centre-of-mass frame).
template <int N>
struct GradKin {
  uint32_t leg[N];
  uint32_t hel;
  double x1, x2, shat, rs;
  double q[N][4];   // RAMBO's q (position order; beam positions unused)
  double Q[4];
  RamboMap map;
  double pc[N][4];  // physical CM momenta, position order
  int ex;           // momentum scale 2^-ex of the recursion
  double sc;
};

// The draws of a workgroup's events in LDS, a row of 4 (N - 2) words each (and a word of padding: the
// rows start in all banks), and their adjoints on the way back.  A lane's words lie together in
// memory and it takes them in the order of its colour ordering: read from there they cost a chain of
// two loads and a line per lane and word, while the workgroup's rows are one contiguous block,
// whose loads depend on nothing (second kernel, when the step was made: n = 8 FP32, 2^20 events
// 332 -> 274 us; n = 6 FP64, 2 10^5 39 -> 34).  Called by every lane of the workgroup.
template <int N>
struct DrawRows {
  static constexpr int W = 4 * (N - 2), kStride = W + 1;
  static constexpr int bytes(int events) { return events * kStride * 8; }
  template <typename F>
  __device__ __forceinline__ static void each(int64_t first, int64_t count, int events, const F& f) {
    const int n = (int)(count - first < events ? count - first : events) * W;
#pragma unroll 8
    for (int w = (int)threadIdx.x; w < n; w += (int)blockDim.x) f(w, w / W * kStride + w % W);
  }
  __device__ __forceinline__ static void load(double* rows, const double* u, int64_t first, int64_t count, int events) {
    each(first, count, events, [&](int w, int slot) { rows[slot] = u[first * W + w]; });
    __syncthreads();
  }
  __device__ __forceinline__ static void store(const double* rows, double* u, int64_t first, int64_t count,
                                               int events) {
    __syncthreads();
    each(first, count, events, [&](int w, int slot) { u[first * W + w] = rows[slot]; });
  }
};

// (row: the event's draws, DrawRows)
template <int N>
__device__ __forceinline__ void grad_front(const GradArgs& G, int64_t i, const double* row, GradKin<N>& K) {
  K.leg[0] = 0;
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const uint32_t l = G.order[i * N + t];
    K.leg[t] = l < 1u ? 1u : (l > (uint32_t)(N - 1) ? (uint32_t)(N - 1) : l);
  }
  K.hel = G.hel[i];
  K.x1 = 1.0;
  K.x2 = 1.0;
  K.shat = G.sqrt_s * G.sqrt_s;
  K.rs = G.sqrt_s;
  if (G.use_pdf) {
    K.x1 = G.x12[2 * i];
    K.x2 = G.x12[2 * i + 1];
    K.shat = K.x1 * K.x2 * G.sqrt_s * G.sqrt_s;
    K.rs = sqrt(K.shat);
  }
  // RAMBO in position order (centre-of-mass frame)
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) K.Q[mu] = 0.0;
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const bool out = K.leg[t] >= 2u;
    const uint32_t pidx = out ? K.leg[t] - 2u : 0u;
    const double* u = row + 4 * pidx;
    rambo_q(u[0], u[1], u[2], u[3], K.q[t]);
    if (out) {
#pragma unroll
      for (int mu = 0; mu < 4; ++mu) K.Q[mu] += K.q[t][mu];
    }
  }
  K.map.init(K.Q, K.rs);
#pragma unroll
  for (int t = 0; t < N; ++t) {
    K.map.apply(K.q[t], K.pc[t]);
    if (K.leg[t] < 2u) {
      const double zs = K.leg[t] == 0u ? 0.5 * K.rs : -0.5 * K.rs;
      K.pc[t][0] = 0.5 * K.rs; K.pc[t][1] = 0.0; K.pc[t][2] = 0.0; K.pc[t][3] = zs;
    }
  }
  double esum = 0.0;
#pragma unroll
  for (int t = 0; t < N; ++t) esum += fabs(K.pc[t][0]);
  K.ex = ilogb(0.5 * esum);
  K.sc = ldexp(1.0, -K.ex);
}

// log w_int from |m|^2 of the scaled momenta; false (and zero gradients written) when
// |m|^2 vanishes or is not finite.
template <int N>
__device__ __forceinline__ bool grad_logw(const GradArgs& G, int64_t i, const GradKin<N>& K, double m2, bool store) {
  const double ln2 = 0.69314718055994530942;
  double lw = log(m2) + (double)(2 * K.ex * (4 - N) - (N - 2)) * ln2 + (N - 5) * log(K.shat) + G.log_const;
  if (G.use_pdf) lw += G.pdf_a * (log(K.x1) + log(K.x2)) + G.pdf_b * (log1p(-K.x1) + log1p(-K.x2));
  if (!(m2 > 0.0) || !isfinite(m2)) {
    if (store) {  // (the second kernel writes the draws' zeros)
      G.grad_x[2 * i] = 0.0;
      G.grad_x[2 * i + 1] = 0.0;
      if (G.logw) G.logw[i] = -INFINITY;
    }
    return false;
  }
  if (store && G.logw) G.logw[i] = lw;
  return true;
}

// From the CM momentum adjoints pb (polarisation adjoints included) and the sqrt(s_hat)
// adjoint of the beams: RAMBO's conformal map, q(rho), and x1, x2; writes the gradient in x1, x2
// and puts that in the draws in their place in row.
template <int N>
__device__ __forceinline__ void grad_back(const GradArgs& G, int64_t i, const GradKin<N>& K, const double (&pb)[N][4],
                                          double rsb, double* row) {
  const double gw = G.gout ? G.gout[i] : 1.0;
  RamboMapAdj A{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  double qb[N][4];
#pragma unroll
  for (int t = 1; t < N; ++t) {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) qb[t][mu] = 0.0;
    if (K.leg[t] >= 2u) rambo_apply_adj(K.map, K.q[t], pb[t], qb[t], A);
  }
  double Qb[4] = {0.0, 0.0, 0.0, 0.0};
  rambo_init_adj(K.map, K.Q, A, Qb, rsb);
  // an ordering is not checked: of a leg that it names twice the last position's adjoint is kept, a leg
  // that it leaves out has none
  uint32_t leg[N], named = 1u;
#pragma unroll
  for (int t = 1; t < N; ++t) {
    leg[t] = K.leg[t];
    named |= 1u << leg[t];
  }
  if (named != (1u << N) - 1u) {
    uint32_t later = 0;
#pragma unroll
    for (int t = N - 1; t >= 1; --t) {
      const uint32_t bit = 1u << leg[t];
      leg[t] = (later & bit) ? 0u : leg[t];
      later |= bit;
    }
    for (int c = 0; c < DrawRows<N>::W; ++c)
      if (!((named >> (c / 4 + 2)) & 1u)) row[c] = 0.0;
  }
#pragma unroll
  for (int t = 1; t < N; ++t) {
    if (leg[t] >= 2u) {
      double* u = row + 4 * (leg[t] - 2u);
      double qbt[4], rb[4];
#pragma unroll
      for (int mu = 0; mu < 4; ++mu) qbt[mu] = qb[t][mu] + Qb[mu];
      rambo_q_adj(u[0], u[1], u[2], u[3], K.q[t][0], qbt, rb);
#pragma unroll
      for (int c = 0; c < 4; ++c) u[c] = gw * rb[c];
    }
  }
  // s_hat = x1 x2 S:  d sqrt(s_hat) / dx_i = sqrt(s_hat) / (2 x_i)
  double xb1 = 0.0, xb2 = 0.0;
  if (G.use_pdf) {
    xb1 = rsb * K.rs / (2.0 * K.x1) + (N - 5) / K.x1 + G.pdf_a / K.x1 - G.pdf_b / (1.0 - K.x1);
    xb2 = rsb * K.rs / (2.0 * K.x2) + (N - 5) / K.x2 + G.pdf_a / K.x2 - G.pdf_b / (1.0 - K.x2);
  }
  G.grad_x[2 * i] = gw * xb1;
  G.grad_x[2 * i + 1] = gw * xb2;
}

// The recursion's adjoints go to the second kernel (k_grad_back), which takes them through
// the helicity sources, the momentum scaling, RAMBO and x1, x2: kept in one kernel, those
// values stay live across the reverse sweep and spill to scratch.  Per position t = 1..N-1
// nine words in the recursion's precision: the contravariant adjoint of the scaled recursion
// momentum (4), then the adjoints of the source's words that are not identically zero, re[1..3],
// im[1], im[2]; then a flag (0: |A|^2 = 0, nothing to do).  Layout [word][event], so
// neighbouring lanes write neighbouring words.  (All eight source words in FP64 took 680 B an
// event at n = 8 instead of 256, which bounded the second kernel.)
template <int N>
struct GradRaw {
  static constexpr int words = grad_words(N), kFlag = words - 1;
  __host__ __device__ static constexpr int at(int t, int w) { return 9 * (t - 1) + w; }
  // word of the source adjoint's component mu, -1 where the source is zero
  __host__ __device__ static constexpr int re(int mu) { return mu == 0 ? -1 : 3 + mu; }
  __host__ __device__ static constexpr int im(int mu) { return mu == 1 || mu == 2 ? 6 + mu : -1; }
};

// One event per lane: forward (CM momenta, recursion), log w_int, reverse sweep, momentum
// adjoints.
template <int N, typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_grad(GradArgs G) {
  constexpr int L = N - 1;
  using SP = Spans<L>;
  extern __shared__ __align__(16) unsigned char gdyn[];  // DrawRows
  double* rows = reinterpret_cast<double*>(gdyn);
  const int64_t first = (int64_t)blockIdx.x * blockDim.x, i = first + threadIdx.x;
  DrawRows<N>::load(rows, G.u, first, G.count, (int)blockDim.x);
  if (i >= G.count) return;
  GradKin<N> K;
  grad_front<N>(G, i, rows + threadIdx.x * DrawRows<N>::kStride, K);
  double k[L][4];
  cv4<T> src[L];
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double sg = K.leg[t] < 2u ? -K.sc : K.sc;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) k[t - 1][mu] = sg * K.pc[t][mu];
    src[t - 1] = polarisation<T>(K.pc[t], (K.hel >> K.leg[t]) & 1u);
  }
  const cv4<T> e0 = polarisation<T>(K.pc[0], K.hel & 1u);
  cv4<T> J[SP::count];
  T Sr[SP::count], Si[SP::count];
  cv4<T> V;
  SpanKLegs<L, T> ks{k};
  bg_forward<L, T>(ks, src, J, Sr, Si, V);
  // bg_forward leaves the span scalars negated; the reverse sweep takes S itself
  static_for<L, SP::count>([&](auto sc) {
    Sr[decltype(sc)::value] = -Sr[decltype(sc)::value];
    Si[decltype(sc)::value] = -Si[decltype(sc)::value];
  });
  T mr, mi;
  cdot(e0, V, mr, mi);
  const double m2 = double(mr) * double(mr) + double(mi) * double(mi);
  using R = GradRaw<N>;
  T* o = static_cast<T*>(G.pbuf) + i;
  if (!grad_logw<N>(G, i, K, m2, true)) {
    o[R::kFlag * G.count] = T(0);  // nothing for the second kernel
    return;
  }
  // reverse sweep: d log|m|^2 / dm = 2 m / |m|^2
  cv4<T> srcb[L], e0b;
  T kb[L][4];
  bg_reverse<L, T>(k, J, Sr, Si, e0, V, T(2.0 * double(mr) / m2), T(2.0 * double(mi) / m2), srcb, e0b, kb);
#pragma unroll
  for (int t = 1; t < N; ++t) {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      o[R::at(t, mu) * G.count] = kb[t - 1][mu];
      if (R::re(mu) >= 0) o[R::at(t, R::re(mu)) * G.count] = srcb[t - 1].re[mu];
      if (R::im(mu) >= 0) o[R::at(t, R::im(mu)) * G.count] = srcb[t - 1].im[mu];
    }
  }
  o[R::kFlag * G.count] = T(1);
}

// Whether the gradient kernel keeps its span scalars distributed over the lanes of a group:
// it holds the currents and their adjoints (twice the forward's registers).
template <int L, int G, typename T>
constexpr bool grad_dist_scalars() {
  return G > 1 && Spans<L>::count * 4 * (4 / G) * (int)(sizeof(T) / 4) > 160;
}

// GL lanes per event (the grouped recursion and its reverse sweep, bg_group_adj.hpp); every
// lane evaluates the kinematics, lane g writes its components of the raw adjoints.  The
// forward values pass an optimisation barrier before the sweep, so the compiler does not keep
// the forward pass's intermediates live across it.  Workgroups of kLdsLanes lanes, with
// grad_lds_bytes of dynamic LDS: the draws' rows, then the span table.  Bound by VALU issue at one wave per SIMD (87% at
// n = 8: 20892 instructions a wave).
// Whether its span momenta and propagators come from the LDS table: where the sweep spills without
// it too, what the table brings into registers spills more than the sums cost (us, sums / table:
// FP64 n = 11, 6 10^4 events 1465 / 1579, n = 12, 8 10^4 3024 / 3408; FP32 n = 12, 10^5 1322 / 1406; where it
// fits, n = 8 FP32, 2^20, this kernel alone 1730 / 1517).
template <int N, typename T>
constexpr bool grad_span_table() { return sizeof(T) == 8 ? N <= 8 : N <= 11; }

template <int N, typename T, int GL>
constexpr int grad_lds_bytes() {
  constexpr int table = grad_span_table<N, T>() ? SpanKGroupLds<N - 1, GL, T>::kBytes * kLdsLanes : 0;
  constexpr int rows = DrawRows<N>::bytes(kLdsLanes / GL);
  return table > rows ? table : rows;
}

template <int N, typename T, int GL>
__global__ __launch_bounds__(kLdsLanes) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_grad_g(GradArgs G) {
  constexpr int L = N - 1, C = 4 / GL;
  using SP = Spans<L>;
  using SS = SpanScalars<L, GL, T, grad_dist_scalars<L, GL, T>()>;
  extern __shared__ __align__(16) unsigned char gdyn[];
  const int event = (int)threadIdx.x / GL, g = (int)threadIdx.x % GL;
  const int64_t first = (int64_t)blockIdx.x * (kLdsLanes / GL), i = first + event;
  DrawRows<N>::load(reinterpret_cast<double*>(gdyn), G.u, first, G.count, kLdsLanes / GL);
  if (i >= G.count) return;
  GradKin<N> K;
  grad_front<N>(G, i, reinterpret_cast<double*>(gdyn) + event * DrawRows<N>::kStride, K);
  __syncthreads();  // the span table takes the rows' place
  const LaneShare<GL, T> ls(g);
  const LaneShare<GL, double> lsd(g);
  double k[L][C];  // covariant, this lane's components
  cvl<T, C> src[L], e0;
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double sg = K.leg[t] < 2u ? -K.sc : K.sc;
#pragma unroll
    for (int c = 0; c < C; ++c) k[t - 1][c] = lsd.sg[c] * (sg * lsd.template pick<true>(K.pc[t], c));
    const cv4<T> e = polarisation<T>(K.pc[t], (K.hel >> K.leg[t]) & 1u);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      src[t - 1].re[c] = ls.template pick<true>(e.re, c);
      src[t - 1].im[c] = ls.template pick<true>(e.im, c);
    }
  }
  {
    const cv4<T> e = polarisation<T>(K.pc[0], K.hel & 1u);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      e0.re[c] = ls.template pick<true>(e.re, c);
      e0.im[c] = ls.template pick<true>(e.im, c);
    }
  }
  const auto ks = [&] {
    if constexpr (grad_span_table<N, T>())
      return SpanKGroupLds<L, GL, T>(k, lsd.sg, gdyn, (int)threadIdx.x, kLdsLanes);
    else
      return SpanKGroup<L, GL, T>{k, lsd.sg};
  }();
  cvl<T, C> J[SP::count];
  SS S(g);
  cvl<T, C> V;
  bg_forward_g<L, GL, T>(ls, ks, src, J, S, V);
  T mr, mi;
  cdot_g<GL>(ls, e0, V, mr, mi);
  const double m2 = double(mr) * double(mr) + double(mi) * double(mi);
  using R = GradRaw<N>;
  T* o = static_cast<T*>(G.pbuf) + i;
  if (!grad_logw<N>(G, i, K, m2, g == 0)) {
    if (g == 0) o[R::kFlag * G.count] = T(0);  // nothing for the second kernel
    return;
  }
  static_for<0, SP::count>([&](auto sc) {
    constexpr int q = decltype(sc)::value;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      opaque(J[q].re[c]);
      opaque(J[q].im[c]);
    }
  });
#pragma unroll
  for (int m = 0; m < SS::kSlots; ++m) {
    opaque(S.re[m]);
    opaque(S.im[m]);
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    opaque(V.re[c]);
    opaque(V.im[c]);
  }
  cvl<T, C> srcb[L], e0b;
  T kb[L][C];
  bg_reverse_g<L, GL, T>(ls, ks, J, S, e0, V, T(2.0 * double(mr) / m2), T(2.0 * double(mi) / m2), srcb, e0b, kb);
  // this lane's components of the raw adjoints (contravariant momentum adjoints), past an
  // optimisation barrier: the compiler sinks the sweep into the branches of the stores otherwise
  // (6 KB of scratch per lane at n = 8)
#pragma unroll
  for (int t = 0; t < L; ++t) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      opaque(kb[t][c]);
      opaque(srcb[t].re[c]);
      opaque(srcb[t].im[c]);
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int mu = g * C + c;
#pragma unroll
    for (int t = 1; t < N; ++t) o[R::at(t, mu) * G.count] = ls.sg[c] * kb[t - 1][c];
    if (mu >= 1) {
#pragma unroll
      for (int t = 1; t < N; ++t) o[R::at(t, 3 + mu) * G.count] = srcb[t - 1].re[c];
    }
    if (mu == 1 || mu == 2) {
#pragma unroll
      for (int t = 1; t < N; ++t) o[R::at(t, 6 + mu) * G.count] = srcb[t - 1].im[c];
    }
  }
  if (g == 0) o[R::kFlag * G.count] = T(1);
}

// Second gradient kernel (one lane per event): from the recursion's adjoints that k_grad or
// k_grad_g left in pbuf, the helicity sources' and momenta's adjoints (CM frame), RAMBO's
// conformal map, q(rho) and x1, x2.  Events with |A|^2 = 0 were completed by the first, but for the
// draws' zeros.  Bound by its 700 B an event (2.5 TB/s) and the FP64 chains: 5141 -> 4292 instructions a
// wave and 680 -> 256 B of adjoints an event, and the rows in LDS: n = 8 FP32 442 -> 298 us per 2^20
// events, n = 6 FP64 46 -> 38 per 2 10^5.  (With products of reciprocals for the rounded quotients 3239
// instructions, 273 and 34 us, and results further from their exact values.)
template <int N, typename T>
__device__ __forceinline__ void grad_back_event(const GradArgs& G, int64_t i, double* row) {
  using R = GradRaw<N>;
  const T* __restrict__ o = static_cast<const T*>(G.pbuf) + i;
  if (o[R::kFlag * G.count] == T(0)) {
#pragma unroll
    for (int c = 0; c < DrawRows<N>::W; ++c) row[c] = 0.0;
    return;
  }
  GradKin<N> K;
  grad_front<N>(G, i, row, K);
  double pb[N][4];
  double rsb = 0.0;
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) pb[0][mu] = 0.0;
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double sg = K.leg[t] < 2u ? -K.sc : K.sc;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) pb[t][mu] = sg * (double)o[R::at(t, mu) * G.count];
    if (K.leg[t] >= 2u) {
      double er[4] = {0.0, 0.0, 0.0, 0.0}, ei[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int mu = 1; mu < 4; ++mu) {
        er[mu] = (double)o[R::at(t, R::re(mu)) * G.count];
        if (R::im(mu) >= 0) ei[mu] = (double)o[R::at(t, R::im(mu)) * G.count];
      }
      polarisation_adj(K.pc[t], (K.hel >> K.leg[t]) & 1u, er, ei, pb[t]);
    } else {
      rsb += 0.5 * (pb[t][0] - pb[t][3]);  // leg 1: p = (rs/2)(1, 0, 0, -1)
    }
  }
  grad_back<N>(G, i, K, pb, rsb, row);
}

// Launch: kLdsLanes lanes, DrawRows<N>::bytes(kLdsLanes) bytes of dynamic LDS.
template <int N, typename T>
__global__ __launch_bounds__(kLdsLanes) __attribute__((amdgpu_waves_per_eu(N <= 8 ? 2 : 1, 8))) void k_grad_back(
    GradArgs G) {
  extern __shared__ __align__(16) unsigned char gdyn[];
  double* rows = reinterpret_cast<double*>(gdyn);
  const int64_t first = (int64_t)blockIdx.x * kLdsLanes, i = first + threadIdx.x;
  DrawRows<N>::load(rows, G.u, first, G.count, kLdsLanes);
  if (i < G.count) grad_back_event<N, T>(G, i, rows + threadIdx.x * DrawRows<N>::kStride);
  DrawRows<N>::store(rows, G.grad_u, first, G.count, kLdsLanes);
}

}  // namespace bgk
