// The recursion of Eqs. 3.1-3.2 and the closure of Eq. 3.6 with one event spread over G
// adjacent lanes of a wave (G = 2 or 4; the one-lane form is bg_amplitude).
//
// Lane g of a group holds the Lorentz components mu = g C .. g C + C - 1 (C = 4 / G) of
// every current and span scalar's share, so a lane needs about 1/G of the registers of
// the one-lane form; at n >= 10 in FP32 and n >= 9 in FP64 the one-lane form exceeds the
// 512 registers a lane can address and spills to scratch memory.  Minkowski products are
// formed per lane over its components with their metric signs sigma_mu = (+,-,-,-) and
// completed across the group by DPP lane permutations; every lane of the group ends with
// the bitwise same total (IEEE addition is commutative), so the group stays consistent.
//
// Span momenta enter covariantly, K_mu = sigma_mu K^mu: the FP64 leg momenta are signed
// once per event, so J.K needs no signs, and the K-dependent part of a bracket is summed
// covariantly and converted to contravariant once per span.  K^2 is the group sum of the
// lanes' FP64 partials sigma_mu K_mu^2.
#pragma once

#include "bg_device.hpp"

namespace bgk {

template <typename T, int C>
struct cvl {
  T re[C], im[C];
};

// DPP quad permutations: swap neighbouring lanes, swap neighbouring lane pairs
constexpr int kDppSwap1 = 0xB1;  // quad_perm [1, 0, 3, 2]
constexpr int kDppSwap2 = 0x4E;  // quad_perm [2, 3, 0, 1]

// (old value 0 with bound_ctrl: the FP32 form folds into v_add_f32_dpp)
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ double dpp_mov(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum over the G lanes of a group; every lane receives the same total.  (Kept apart from
// neighbouring products so that the FP32 add takes its operand through DPP.)
template <int G, typename T>
__device__ __forceinline__ T group_sum(T x) {
#pragma clang fp contract(off)
  if constexpr (G >= 2) x = x + dpp_mov<kDppSwap1>(x);
  if constexpr (G >= 4) x = x + dpp_mov<kDppSwap2>(x);
  return x;
}

// This lane's share of a group: its first component and the metric signs of its components.
template <int G, typename T>
struct LaneShare {
  static constexpr int C = 4 / G;
  int mu0;     // first component held
  T sg[C];     // sigma of each held component
  __device__ __forceinline__ explicit LaneShare(int g) : mu0(g * C) {
#pragma unroll
    for (int c = 0; c < C; ++c) sg[c] = c == 0 && mu0 == 0 ? T(1) : T(-1);  // only the first varies
  }
  // the held components of a full four-vector, without dynamic register indexing: one select
  // for two lanes in the forward kernels; bit masks for four lanes, and for two in the
  // gradient kernels (BITS), where selects between elements of one array are turned back into
  // a dynamically indexed array on the stack
  template <bool BITS = false, typename U>
  __device__ __forceinline__ U pick(const U (&v)[4], int c) const {
    if constexpr (G == 4 || BITS) {
      using B = typename std::conditional<sizeof(U) == 8, uint64_t, uint32_t>::type;
      B r = 0;
#pragma unroll
      for (int q = 0; q < G; ++q) r |= __builtin_bit_cast(B, v[q * C + c]) & (B)(-(B)(mu0 == q * C));
      return __builtin_bit_cast(U, r);
    } else {
      U r = v[c];
#pragma unroll
      for (int q = 1; q < G; ++q) r = (mu0 == q * C) ? v[q * C + c] : r;
      return r;
    }
  }
};

// DPP control that gives every lane of a group of G adjacent lanes the value of the group's
// lane K (a quad permutation: [K, K, K, K] for G = 4, [K, K, 2 + K, 2 + K] for G = 2).
template <int G, int K>
constexpr int group_bcast_ctrl() {
  return G == 4 ? (K | (K << 2) | (K << 4) | (K << 6)) : (K | (K << 2) | ((2 + K) << 4) | ((2 + K) << 6));
}

template <int G, int K, typename T>
__device__ __forceinline__ T group_bcast(T x) {
  if constexpr (G == 1) {
    return x;
  } else if constexpr (std::is_same<T, float>::value) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), group_bcast_ctrl<G, K>(),
                                                              0xF, 0xF, false));
  } else {
    return dpp_mov<group_bcast_ctrl<G, K>()>(x);
  }
}

// Whether a group keeps its span scalars distributed over its lanes: where the currents of
// every span already take most of a lane's registers (FP32 n = 12 with two lanes), replicating
// the scalars on every lane would spill.
template <int L, int G, typename T>
constexpr bool dist_scalars() {
  return G > 1 && Spans<L>::count * 2 * (4 / G) * (int)(sizeof(T) / 4) > 240;
}

// The span scalars S of a group (the complex sums of the three-gluon dots, one per span of
// two or more legs; spans counted from the first of two legs, q = s - L).  Replicated: every
// lane holds every scalar.  Distributed: lane q % G of the group holds span q in slot q / G,
// and a read broadcasts it over the group (one DPP move per word); writes of a group-uniform
// value go to the owning lane by a select.  Either way every lane reads bitwise the value
// that was written.
template <int L, int G, typename T, bool DIST = dist_scalars<L, G, T>()>
struct SpanScalars {
  static constexpr int kCount = Spans<L>::count - L;
  static constexpr int kSlots = DIST ? (kCount + G - 1) / G : kCount;
  T re[kSlots], im[kSlots];
  int g;  // this lane's place in its group
  __device__ __forceinline__ explicit SpanScalars(int g_) : g(g_) {}
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int m = 0; m < kSlots; ++m) re[m] = im[m] = T(0);
  }
  template <int S>
  __device__ __forceinline__ void get(T& r, T& i) const {
    constexpr int q = S - L;
    static_assert(q >= 0 && q < kCount, "span scalar index");
    if constexpr (DIST) {
      r = group_bcast<G, q % G>(re[q / G]);
      i = group_bcast<G, q % G>(im[q / G]);
    } else {
      r = re[q];
      i = im[q];
    }
  }
  template <int S>
  __device__ __forceinline__ void put(T r, T i) {
    constexpr int q = S - L;
    static_assert(q >= 0 && q < kCount, "span scalar index");
    if constexpr (DIST) {
      const bool own = g == q % G;
      re[q / G] = own ? r : re[q / G];
      im[q / G] = own ? i : im[q / G];
    } else {
      re[q] = r;
      im[q] = i;
    }
  }
  // S -= (r, i) for a group-uniform (r, i)
  template <int S>
  __device__ __forceinline__ void sub(T r, T i) {
    constexpr int q = S - L;
    static_assert(q >= 0 && q < kCount, "span scalar index");
    if constexpr (DIST) {
      const bool own = g == q % G;
      re[q / G] = own ? re[q / G] - r : re[q / G];
      im[q / G] = own ? im[q / G] - i : im[q / G];
    } else {
      re[q] -= r;
      im[q] -= i;
    }
  }
};

// x.y over the group (bilinear, metric (+,-,-,-))
template <int G, typename T, int C>
__device__ __forceinline__ void cdot_g(const LaneShare<G, T>& ls, const cvl<T, C>& x, const cvl<T, C>& y, T& r,
                                       T& i) {
  r = ls.sg[0] * fmac(-x.im[0], y.im[0], x.re[0] * y.re[0]);
  i = ls.sg[0] * fmac(x.im[0], y.re[0], x.re[0] * y.im[0]);
#pragma unroll
  for (int c = 1; c < C; ++c) {
    r = fmac(ls.sg[c], fmac(-x.im[c], y.im[c], x.re[c] * y.re[c]), r);
    i = fmac(ls.sg[c], fmac(x.im[c], y.re[c], x.re[c] * y.im[c]), i);
  }
  r = group_sum<G>(r);
  i = group_sum<G>(i);
}

// x.K over the group for a covariant real K (this lane's components)
template <int G, typename T, int C>
__device__ __forceinline__ void rdot_g(const cvl<T, C>& x, const T (&k)[C], T& r, T& i) {
  r = x.re[0] * k[0];
  i = x.im[0] * k[0];
#pragma unroll
  for (int c = 1; c < C; ++c) {
    r = fmac(x.re[c], k[c], r);
    i = fmac(x.im[c], k[c], i);
  }
  r = group_sum<G>(r);
  i = group_sum<G>(i);
}

template <typename T, int C>
__device__ __forceinline__ void caxpy_l(T cr, T ci, const cvl<T, C>& y, cvl<T, C>& acc) {
#pragma unroll
  for (int c = 0; c < C; ++c) {
    acc.re[c] = fmac(-ci, y.im[c], fmac(cr, y.re[c], acc.re[c]));
    acc.im[c] = fmac(ci, y.re[c], fmac(cr, y.im[c], acc.im[c]));
  }
}

// Covariant span momenta of this lane's components, summed left to right in FP64 over the
// legs and cast to T; propagators 1/K^2 from the group sum of FP64 partials (the gradients of the
// largest n, grad_span_table).
template <int L, int G, typename T>
struct SpanKGroup {
  static constexpr int C = 4 / G;
  const double (&k)[L][C];   // covariant FP64 leg components held by this lane
  const double (&sg)[C];     // their metric signs
  // Every use sums afresh: an optimisation barrier on the first term keeps the compiler from merging
  // the sums of one span over the whole kernel and holding them in registers.
  template <int A, int B>
  __device__ __forceinline__ void sum(double d[C]) const {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      d[c] = k[A][c];
      opaque(d[c]);
    }
    static_for<A + 1, B + 1>([&](auto t) {
#pragma unroll
      for (int c = 0; c < C; ++c) d[c] += k[decltype(t)::value][c];
    });
  }
  template <int A, int B>
  __device__ __forceinline__ void K(T (&out)[C]) const {
    double d[C];
    sum<A, B>(d);
#pragma unroll
    for (int c = 0; c < C; ++c) out[c] = T(d[c]);
  }
  template <int A, int B>
  __device__ __forceinline__ T prop() const {
    double d[C];
    sum<A, B>(d);
    double part;
    {
#pragma clang fp contract(off)
      part = sg[0] * (d[0] * d[0]);
#pragma unroll
      for (int c = 1; c < C; ++c) part = part + sg[c] * (d[c] * d[c]);
    }
    const double k2 = group_sum<G>(part);
    if constexpr (std::is_same<T, float>::value)
      return __builtin_amdgcn_rcpf(float(k2));
    else
      return 1.0 / k2;
  }
};

// Covariant span momenta and propagators, read from a per-workgroup LDS table filled once per
// event: for every span of 2..L-1 legs this lane's components, summed left to right in FP64 over
// its legs and cast to T, and 1/K^2 from the group sum of the FP64 partials.  Layout [span][lane]
// of C components, so that a wave's reads are contiguous, then the propagators, one per group: G
// spans to a row.  One table read replaces the FP64 sums and conversions at every use, and nothing
// of them stays live in registers but the legs in T.  (The propagators too: formed at their use
// they keep the FP64 legs live.  Without / with, and with the unit's scheduler choice: FP32
// n = 12 2.09 / 2.01 ms per 2^20 events; the gradient's n = 8 kernel, where the sums were formed
// at every use, 1730 / 1517 us per 2^20.)
template <int L, int G, typename T>
struct SpanKGroupLds {
  static constexpr int C = 4 / G;
  static constexpr int kSpans = Spans<L>::count - L - 1;  // spans of 2..L-1 legs
  static constexpr int kBytes = kSpans * C * (int)sizeof(T) + (kSpans + G - 1) / G * (int)sizeof(T);  // per lane
  struct alignas(C * sizeof(T)) Row {
    T v[C];
  };
  Row* kt;    // &table[0][lane]
  T* pt;      // &props[0][first lane of the group]
  int lanes;  // lanes per workgroup (the row stride)
  T leg[L][C];
  __device__ __forceinline__ SpanKGroupLds(const double (&k)[L][C], const double (&sg)[C], unsigned char* lds, int lane,
                                           int lanes_)
      : kt(reinterpret_cast<Row*>(lds) + lane),
        pt(reinterpret_cast<T*>(reinterpret_cast<Row*>(lds) + kSpans * lanes_) + (lane - lane % G)),
        lanes(lanes_) {
    using SP = Spans<L>;
    static_for<0, L>([&](auto ac) {
      constexpr int a = decltype(ac)::value;
      double acc[C];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        acc[c] = k[a][c];
        leg[a][c] = T(acc[c]);
      }
      static_for<a + 1, L>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        if constexpr (b - a + 1 < L) {
          constexpr int q = SP::at(a, b) - L;
          Row r;
#pragma unroll
          for (int c = 0; c < C; ++c) {
            acc[c] += k[b][c];
            r.v[c] = T(acc[c]);
          }
          kt[q * lanes] = r;
          double part;
          {
#pragma clang fp contract(off)
            part = sg[0] * (acc[0] * acc[0]);
#pragma unroll
            for (int c = 1; c < C; ++c) part = part + sg[c] * (acc[c] * acc[c]);
          }
          const double k2 = group_sum<G>(part);
          T prop;
          if constexpr (std::is_same<T, float>::value)
            prop = __builtin_amdgcn_rcpf(float(k2));
          else
            prop = 1.0 / k2;
          pt[q / G * lanes + q % G] = prop;  // every lane of the group writes the same
        }
      });
    });
    // the recursion reads the table back instead of keeping the values in registers
    asm volatile("" ::: "memory");
  }
  template <int A, int B>
  __device__ __forceinline__ void K(T (&out)[C]) const {
    if constexpr (A == B) {
#pragma unroll
      for (int c = 0; c < C; ++c) out[c] = leg[A][c];
    } else {
      constexpr int q = Spans<L>::at(A, B) - L;
      static_assert(q >= 0 && q < kSpans, "span of 2..L-1 legs");
      const Row r = kt[q * lanes];
#pragma unroll
      for (int c = 0; c < C; ++c) out[c] = r.v[c];
    }
  }
  template <int A, int B>
  __device__ __forceinline__ T prop() const {
    constexpr int q = Spans<L>::at(A, B) - L;
    return pt[q / G * lanes + q % G];
  }
};

// One span [A..B]: its bracket sum V (contravariant, this lane's components).
template <int L, int A, int B, int G, typename T, typename KS, typename SS>
__device__ __forceinline__ void span_vertex_g(const LaneShare<G, T>& ls, const KS& ks,
                                              const cvl<T, 4 / G> (&J)[Spans<L>::count], const SS& S,
                                              cvl<T, 4 / G>& V, T& sr, T& si) {
  constexpr int C = 4 / G;
  using SP = Spans<L>;
  cvl<T, C> X, Z, Yc;  // (J.K) J terms, S terms (contravariant); d (K_A - K_B) (covariant)
#pragma unroll
  for (int c = 0; c < C; ++c) X.re[c] = X.im[c] = Z.re[c] = Z.im[c] = Yc.re[c] = Yc.im[c] = T(0);
  sr = T(0);
  si = T(0);
  static_for<A, B>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr int PA = SP::at(A, i), PB = SP::at(i + 1, B);
    T ka[C], kb[C];
    ks.template K<A, i>(ka);
    ks.template K<i + 1, B>(kb);
    T dr, di, ar, ai, br, bi;
    cdot_g<G>(ls, J[PA], J[PB], dr, di);
    rdot_g<G>(J[PA], kb, ar, ai);
    rdot_g<G>(J[PB], ka, br, bi);
    caxpy_l(ar, ai, J[PB], X);
    caxpy_l(-br, -bi, J[PA], X);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const T dk = ka[c] - kb[c];
      Yc.re[c] = fmac(dr, dk, Yc.re[c]);
      Yc.im[c] = fmac(di, dk, Yc.im[c]);
    }
    sr += dr;
    si += di;
  });
  static_for<A, B - 1>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    static_for<i + 1, B>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      T dr, di;
      cdot_g<G>(ls, J[SP::at(A, i)], J[SP::at(j + 1, B)], dr, di);
      caxpy_l(dr, di, J[SP::at(i + 1, j)], X);
    });
  });
  static_for<A + 1, B>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    T r, i;
    S.template get<SP::at(A, j)>(r, i);
    caxpy_l(-r, -i, J[SP::at(j + 1, B)], Z);
  });
  static_for<A, B - 1>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    T r, im;
    S.template get<SP::at(i + 1, B)>(r, im);
    caxpy_l(-r, -im, J[SP::at(A, i)], Z);
  });
#pragma unroll
  for (int c = 0; c < C; ++c) {
    V.re[c] = fmac(T(2), X.re[c], fmac(ls.sg[c], Yc.re[c], Z.re[c]));
    V.im[c] = fmac(T(2), X.im[c], fmac(ls.sg[c], Yc.im[c], Z.im[c]));
  }
}

// Forward recursion: every stored current and span scalar, and the undivided bracket sum V
// of the full span (this lane's components).
template <int L, int G, typename T, typename KS, typename SS>
__device__ __forceinline__ void bg_forward_g(const LaneShare<G, T>& ls, const KS& ks,
                                             const cvl<T, 4 / G> (&src)[L], cvl<T, 4 / G> (&J)[Spans<L>::count],
                                             SS& S, cvl<T, 4 / G>& Vfull) {
  constexpr int C = 4 / G;
  using SP = Spans<L>;
  static_for<0, L>([&](auto ac) { J[decltype(ac)::value] = src[decltype(ac)::value]; });
  static_for<2, L>([&](auto lc) {
    constexpr int len = decltype(lc)::value;
    static_for<0, L - len + 1>([&](auto ac) {
      constexpr int a = decltype(ac)::value, b = a + len - 1, s = SP::at(a, b);
      cvl<T, C> V;
      T sr, si;
      span_vertex_g<L, a, b, G, T>(ls, ks, J, S, V, sr, si);
      const T prop = ks.template prop<a, b>();
#pragma unroll
      for (int c = 0; c < C; ++c) {
        J[s].re[c] = V.re[c] * prop;
        J[s].im[c] = V.im[c] * prop;
      }
      S.template put<s>(sr, si);
    });
  });
  T sr, si;
  span_vertex_g<L, 0, L - 1, G, T>(ls, ks, J, S, Vfull, sr, si);
}

// Forward recursion and closure m = eps0 . V[0..L-1] (every lane of the group gets m).
template <int L, int G, typename T, typename KS>
__device__ __forceinline__ void bg_amplitude_g(const LaneShare<G, T>& ls, const KS& ks,
                                               const cvl<T, 4 / G> (&src)[L], const cvl<T, 4 / G>& eps0,
                                               double& m_re, double& m_im) {
  constexpr int C = 4 / G;
  using SP = Spans<L>;
  cvl<T, C> J[SP::count];
  SpanScalars<L, G, T> S(ls.mu0 / C);
  cvl<T, C> V;
  bg_forward_g<L, G, T>(ls, ks, src, J, S, V);
  T mr, mi;
  cdot_g<G>(ls, eps0, V, mr, mi);
  m_re = double(mr);
  m_im = double(mi);
}

// ----------------------------------------------------------------------------------------
// FP64 with an event on a pair of lanes (n >= 6; n = 7, 8 in short calls).  What limits these classes is where a lane
// keeps its currents (n = 12: 498 registers of 512), so, as in the one-lane FP64 form
// (bg_amplitude_d), the covariant leg momenta and the span scalars -S/2 live in LDS and brackets
// accumulate V / 2 in one vector.  Lane 0 holds the components (0, 1), lane 1 (3, 2): the first
// slot of a source then has a zero imaginary part on both lanes (LX, LY: leaf operands), the
// second slot the metric sign -1 on both, and only the first slot's sign (+, -) differs.
// Generation, 2^18 events: n = 9 313 -> 272 us, n = 10 (four lanes before) 576 -> 433 us.
// ----------------------------------------------------------------------------------------
struct cvp {
  double re[2], im[2];
};

// LDS per lane: legs [L][lane] as (K_first, K_second), then scalars [span][lane] with the real part
// in the pair's even lane and the imaginary part in its odd one.
template <int L>
constexpr int pair_lds_bytes() { return 16 * L + 8 * (Spans<L>::count - L - 1); }

template <int L>
struct PairSpan {
  double2* leg;      // &leg[0][lane]
  double* sc;        // &sc[0][lane]
  const double2* rd; // &sc[0][lane & ~1], the pair's scalar
  int lanes;         // lanes per workgroup (row stride)
  double sg;         // metric sign of the first slot
  int g;             // lane of the pair
  __device__ __forceinline__ PairSpan(unsigned char* lds, int lane, int lanes_)
      : leg(reinterpret_cast<double2*>(lds) + lane),
        sc(reinterpret_cast<double*>(lds + 16 * L * lanes_) + lane),
        rd(reinterpret_cast<const double2*>(lds + 16 * L * lanes_) + (lane >> 1)),
        lanes(lanes_),
        sg((lane & 1) ? -1.0 : 1.0),
        g(lane & 1) {}
  template <int A>
  __device__ __forceinline__ void add(double (&K)[2]) const {
    const double2 k = leg[A * lanes];
    K[0] += k.x;
    K[1] += k.y;
  }
  // legs A..B summed left to right
  template <int A, int B>
  __device__ __forceinline__ void sum(double (&K)[2]) const {
    const double2 k = leg[A * lanes];
    K[0] = k.x;
    K[1] = k.y;
    static_for<A + 1, B + 1>([&](auto t) { add<decltype(t)::value>(K); });
  }
  template <int S>
  __device__ __forceinline__ void put_scalar(double r, double i) const { sc[(S - L) * lanes] = g ? i : r; }
  template <int S>
  __device__ __forceinline__ double2 scalar() const { return rd[(S - L) * (lanes / 2)]; }
};

// x . y over the pair; xs: x with the first slot times its metric sign (pair_signed)
template <bool LX, bool LY>
__device__ __forceinline__ void pdot(const cvp& xs, const cvp& y, double& r, double& i) {
#pragma clang fp contract(off)
  r = xs.re[0] * y.re[0];
  r = fmac(-xs.re[1], y.re[1], r);
  r = fmac(xs.im[1], y.im[1], r);
  i = -xs.re[1] * y.im[1];
  i = fmac(-xs.im[1], y.re[1], i);
  if constexpr (!LX && !LY) r = fmac(-xs.im[0], y.im[0], r);
  if constexpr (!LY) i = fmac(xs.re[0], y.im[0], i);
  if constexpr (!LX) i = fmac(xs.im[0], y.re[0], i);
  r = group_sum<2>(r);
  i = group_sum<2>(i);
}

// x . K over the pair for a covariant real K
template <bool LX>
__device__ __forceinline__ void prdot(const cvp& x, const double (&k)[2], double& r, double& i) {
#pragma clang fp contract(off)
  r = group_sum<2>(fmac(x.re[1], k[1], x.re[0] * k[0]));
  if constexpr (LX)
    i = group_sum<2>(x.im[1] * k[1]);
  else
    i = group_sum<2>(fmac(x.im[1], k[1], x.im[0] * k[0]));
}

template <bool LY>
__device__ __forceinline__ void paxpy(double cr, double ci, const cvp& y, cvp& acc) {
  acc.re[0] = fmac(cr, y.re[0], acc.re[0]);
  acc.im[0] = fmac(ci, y.re[0], acc.im[0]);
  if constexpr (!LY) {
    acc.re[0] = fmac(-ci, y.im[0], acc.re[0]);
    acc.im[0] = fmac(cr, y.im[0], acc.im[0]);
  }
  acc.re[1] = fmac(-ci, y.im[1], fmac(cr, y.re[1], acc.re[1]));
  acc.im[1] = fmac(ci, y.re[1], fmac(cr, y.im[1], acc.im[1]));
}

template <bool LX>
__device__ __forceinline__ cvp pair_signed(double sg, const cvp& x) {
  cvp s = x;
  s.re[0] = sg * x.re[0];
  if constexpr (!LX) s.im[0] = sg * x.im[0];
  return s;
}

// Half the bracket sum of span [A..B] and its -S/2 (in the order of span_vertex_d, but for the pairs beside
// their left current's brackets from n = 9); KP: the span's momentum.
template <int L, int A, int B>
__device__ __forceinline__ void span_vertex_p(const PairSpan<L>& ks, const cvp (&J)[Spans<L>::count],
                                              double (&KP)[2], cvp& X, double& sr, double& si) {
#pragma clang fp contract(off)
  using SP = Spans<L>;
#pragma unroll
  for (int c = 0; c < 2; ++c) X.re[c] = X.im[c] = 0.0;
  sr = 0.0;
  si = 0.0;
  constexpr bool kApart = L == 6 || L == 7;  // n = 7, 8: the order of span_vertex_pairs
  if constexpr (kApart)
    static_for<A, B - 1>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const cvp xs = pair_signed<i == A>(ks.sg, J[SP::at(A, i)]);
      static_for<i + 1, B>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        double er, ei;
        pdot<i == A, j + 1 == B>(xs, J[SP::at(j + 1, B)], er, ei);
        paxpy<i + 1 == j>(er, ei, J[SP::at(i + 1, j)], X);
      });
    });
  static_for<A + 1, B>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    const double2 c = ks.template scalar<SP::at(A, j)>();
    paxpy<j + 1 == B>(c.x, c.y, J[SP::at(j + 1, B)], X);
  });
  static_for<A, B - 1>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const double2 c = ks.template scalar<SP::at(i + 1, B)>();
    paxpy<i == A>(c.x, c.y, J[SP::at(A, i)], X);
  });
  const double hsg = 0.5 * ks.sg;
  double ka[2];
  static_for<A, B>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr int PA = SP::at(A, i), PB = SP::at(i + 1, B);
    constexpr bool LA = i == A, LB = i + 1 == B;  // leaves
    double kb[2];
    if constexpr (i == A)
      ks.template sum<A, A>(ka);
    else
      ks.template add<i>(ka);
    ks.template sum<i + 1, B>(kb);
    const cvp xs = pair_signed<LA>(ks.sg, J[PA]);
    double dr, di, ar, ai, br, bi;
    pdot<LA, LB>(xs, J[PB], dr, di);
    prdot<LA>(J[PA], kb, ar, ai);
    prdot<LB>(J[PB], ka, br, bi);
    paxpy<LB>(ar, ai, J[PB], X);
    paxpy<LA>(-br, -bi, J[PA], X);
    const double d0 = hsg * (ka[0] - kb[0]), d1 = 0.5 * (kb[1] - ka[1]);
    X.re[0] = fmac(dr, d0, X.re[0]);
    X.im[0] = fmac(di, d0, X.im[0]);
    X.re[1] = fmac(dr, d1, X.re[1]);
    X.im[1] = fmac(di, d1, X.im[1]);
    sr = fmac(-0.5, dr, sr);
    si = fmac(-0.5, di, si);
    // the four-gluon pairs of this left current
    if constexpr (!kApart)
      static_for<i + 1, B>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        double er, ei;
        pdot<LA, j + 1 == B>(xs, J[SP::at(j + 1, B)], er, ei);
        paxpy<i + 1 == j>(er, ei, J[SP::at(i + 1, j)], X);
      });
  });
  ks.template add<B>(ka);
  KP[0] = ka[0];
  KP[1] = ka[1];
}

template <int L>
__device__ __forceinline__ void bg_amplitude_p(const PairSpan<L>& ks, const cvp (&src)[L], const cvp& eps0,
                                               double& m_re, double& m_im) {
  using SP = Spans<L>;
  cvp J[SP::count];
  static_for<0, L>([&](auto ac) { J[decltype(ac)::value] = src[decltype(ac)::value]; });
  static_for<2, L>([&](auto lc) {
    constexpr int len = decltype(lc)::value;
    static_for<0, L - len + 1>([&](auto ac) {
      constexpr int a = decltype(ac)::value, b = a + len - 1, s = SP::at(a, b);
      asm volatile("" ::: "memory");  // momenta and scalars are read afresh in every span
      cvp X;
      double sr, si, K[2];
      span_vertex_p<L, a, b>(ks, J, K, X, sr, si);
      double part;
      {
#pragma clang fp contract(off)
        part = ks.sg * (K[0] * K[0]) - K[1] * K[1];
      }
      const double prop = 2.0 / group_sum<2>(part);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        J[s].re[c] = X.re[c] * prop;
        J[s].im[c] = X.im[c] * prop;
      }
      ks.template put_scalar<s>(sr, si);
    });
  });
  asm volatile("" ::: "memory");
  cvp X;
  double sr, si, K[2], mr, mi;
  span_vertex_p<L, 0, L - 1>(ks, J, K, X, sr, si);
  pdot<true, false>(pair_signed<true>(ks.sg, eps0), X, mr, mi);
  m_re = 2.0 * mr;
  m_im = 2.0 * mi;
}

// ----------------------------------------------------------------------------------------
// FP64 with an event on four lanes (n >= 10 as bg_set_lanes names it), one Lorentz component per
// lane.  Three quarters of a product's instructions would be its cross-lane sum (by DPP two moves
// and an add per step and part: twelve for four multiply-adds), so the sums run on the matrix
// cores: with A constant over its rows, D = A B of v_mfma_f64_4x4x4 gives every lane of a column
// sum_k A_k B_k over the column's four lanes, the metric or plain ones in A.  Each costs four
// issue slots (measured: 16.5 cycles, 32 to its result, no overlap with FP64 vector work) in place
// of six.  Its columns are the lanes l, l + 16, l + 32, l + 48: lane 16 c + e holds component c of
// event e of the wave.  Generation, 2^18 events, with the sums by DPP, scalars and momenta in
// registers and one wave per SIMD: n = 11 819 -> 598 us, n = 12 1172 -> 868 us.  The instruction
// ignores the execution mask, so every lane of a wave runs the recursion (callers clamp the event
// index).  No element of A is zero: a column's infinities and NaN stay its own.
// ----------------------------------------------------------------------------------------
struct cvq {
  double re, im;
};

__device__ __forceinline__ double quad_sum(double a, double x) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, x, 0.0, 0, 0, 0);
}

// LDS per wave: legs [L][lane], then scalars [span][event] as (re, im)
template <int L>
constexpr int quad_lds_bytes() { return 64 * 8 * L + 16 * 16 * (Spans<L>::count - L - 1); }

template <int L>
struct QuadSpan {
  double* leg;   // &leg[0][lane], covariant
  double* put;   // this lane's part of scalar 0
  const double2* get;
  double sg;     // metric sign of the lane's component
  int c;         // component
  __device__ __forceinline__ QuadSpan(unsigned char* lds, int lane)
      : leg(reinterpret_cast<double*>(lds) + lane),
        put(reinterpret_cast<double*>(lds + 64 * 8 * L) + 2 * (lane & 15) + ((lane >> 4) & 1)),
        get(reinterpret_cast<const double2*>(lds + 64 * 8 * L) + (lane & 15)),
        sg(lane < 16 ? 1.0 : -1.0),
        c(lane >> 4) {}
  template <int A, int B>
  __device__ __forceinline__ double sum() const {
    double k = leg[A * 64];
    static_for<A + 1, B + 1>([&](auto t) { k += leg[decltype(t)::value * 64]; });
    return k;
  }
  // (components 2, 3 write what 0, 1 write)
  template <int S>
  __device__ __forceinline__ void put_scalar(double r, double i) const { put[(S - L) * 32] = (c & 1) ? i : r; }
  template <int S>
  __device__ __forceinline__ double2 scalar() const { return get[(S - L) * 16]; }
  // x . y times scale
  __device__ __forceinline__ void dot(const cvq& x, const cvq& y, double& r, double& i, double scale = 1.0) const {
    r = quad_sum(scale * sg, fmac(-x.im, y.im, x.re * y.re));
    i = quad_sum(scale * sg, fmac(x.im, y.re, x.re * y.im));
  }
  __device__ __forceinline__ void rdot(const cvq& x, double k, double& r, double& i) const {
    r = quad_sum(1.0, x.re * k);
    i = quad_sum(1.0, x.im * k);
  }
};

__device__ __forceinline__ void qaxpy(double cr, double ci, const cvq& y, cvq& acc) {
  acc.re = fmac(-ci, y.im, fmac(cr, y.re, acc.re));
  acc.im = fmac(ci, y.re, fmac(cr, y.im, acc.im));
}

// Half the bracket sum of span [A..B] and its -S/2 (as span_vertex_p); KP: the span's momentum.
template <int L, int A, int B>
__device__ __forceinline__ void span_vertex_q(const QuadSpan<L>& ks, const cvq (&J)[Spans<L>::count], double& KP, cvq& X,
                                              double& sr, double& si) {
#pragma clang fp contract(off)
  using SP = Spans<L>;
  X.re = X.im = sr = si = 0.0;
  static_for<A + 1, B>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    const double2 s = ks.template scalar<SP::at(A, j)>();
    qaxpy(s.x, s.y, J[SP::at(j + 1, B)], X);
  });
  static_for<A, B - 1>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const double2 s = ks.template scalar<SP::at(i + 1, B)>();
    qaxpy(s.x, s.y, J[SP::at(A, i)], X);
  });
  double ka = 0.0;
  static_for<A, B>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr int PA = SP::at(A, i), PB = SP::at(i + 1, B);
    ka = i == A ? ks.template sum<A, A>() : ka + ks.template sum<i, i>();
    const double kb = ks.template sum<i + 1, B>();
    double dr, di, ar, ai, br, bi;
    ks.dot(J[PA], J[PB], dr, di, 0.5);
    ks.rdot(J[PA], kb, ar, ai);
    ks.rdot(J[PB], ka, br, bi);
    const double dk = ks.sg * (ka - kb);
    X.re = fmac(dr, dk, X.re);
    X.im = fmac(di, dk, X.im);
    sr -= dr;
    si -= di;
    // the four-gluon pairs of this left current; each sum is used one product after it was
    // issued, so that its latency is covered in the order written (the unit is built without the
    // pre-RA scheduler)
    double er = 0.0, ei = 0.0;
    static_for<i + 1, B>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      double nr, ni;
      ks.dot(J[PA], J[SP::at(j + 1, B)], nr, ni);
      if constexpr (j == i + 1) {
        qaxpy(ar, ai, J[PB], X);
        qaxpy(-br, -bi, J[PA], X);
      } else {
        qaxpy(er, ei, J[SP::at(i + 1, j - 1)], X);
      }
      er = nr;
      ei = ni;
    });
    if constexpr (i + 1 < B) {
      qaxpy(er, ei, J[SP::at(i + 1, B - 1)], X);
    } else {
      qaxpy(ar, ai, J[PB], X);
      qaxpy(-br, -bi, J[PA], X);
    }
  });
  KP = ka + ks.template sum<B, B>();
}

template <int L>
__device__ __forceinline__ void bg_amplitude_q(const QuadSpan<L>& ks, const cvq (&src)[L], const cvq& eps0,
                                               double& m_re, double& m_im) {
  using SP = Spans<L>;
  cvq J[SP::count];
  static_for<0, L>([&](auto ac) { J[decltype(ac)::value] = src[decltype(ac)::value]; });
  static_for<2, L>([&](auto lc) {
    constexpr int len = decltype(lc)::value;
    static_for<0, L - len + 1>([&](auto ac) {
      constexpr int a = decltype(ac)::value, b = a + len - 1, s = SP::at(a, b);
      asm volatile("" ::: "memory");  // momenta and scalars are read afresh in every span
      cvq X;
      double sr, si;
      double K;
      span_vertex_q<L, a, b>(ks, J, K, X, sr, si);
      const double prop = 2.0 / quad_sum(ks.sg, K * K);
      J[s].re = X.re * prop;
      J[s].im = X.im * prop;
      ks.template put_scalar<s>(sr, si);
    });
  });
  asm volatile("" ::: "memory");
  cvq X;
  double sr, si, K, mr, mi;
  span_vertex_q<L, 0, L - 1>(ks, J, K, X, sr, si);
  ks.dot(eps0, X, mr, mi);
  m_re = 2.0 * mr;
  m_im = 2.0 * mi;
}

}  // namespace bgk
