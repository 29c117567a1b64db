// Kernels of the event path: one event per lane, everything for that event kept in the
// lane's registers.  Instantiated per multiplicity N (4..12) and recursion precision T.
#pragma once

#include <type_traits>

#include "bg_device.hpp"
#include "bg_group.hpp"
#include "bg_launch.hpp"
#include "bg_params.hpp"

namespace bgk {

// One event's kinematics: the centre-of-mass momenta in recursion-position order (position 0
// is leg 0, position t >= 1 is leg nib(A, t-1)) for the recursion, and the lab momenta of
// the outgoing gluons in leg order for the cuts and outputs.
template <int N>
struct EventKin {
  double pc[N][4];      // partonic centre-of-mass momenta (RAMBO frame), position order
  double pl[N - 2][4];  // lab momenta of the outgoing legs 2..N-1, leg order
  uint32_t leg[N];      // leg at each position
  uint32_t hel;
  double x1, x2, shat;
};

// Per-lane LDS column through which the outgoing momenta go from leg order to position
// order: slot (4 p + mu) of lane l at perm[(4 p + mu) * stride + l].  Each lane reads only
// what it wrote, so no barrier is needed.
struct PermLds {
  double* col;  // &perm[0][lane]
  int stride;
};

// The column in the kernel's dynamic LDS (launched with perm_lds_bytes(N, blockDim) bytes).
__device__ __forceinline__ PermLds dyn_perm() {
  extern __shared__ double perm_dyn[];
  return PermLds{perm_dyn + threadIdx.x, (int)blockDim.x};
}

// Builds an event's phase-space point (Sec. 3: RAMBO then the longitudinal boost) from
// Philox draws or from caller inputs; writes the optional draw outputs when store is set.
// RAMBO runs over the outgoing legs in leg order (fixed indices, no work for the beams);
// their CM momenta reach the recursion positions through the lane's LDS column.
template <int N>
__device__ __forceinline__ void build_event(const GenClass& C, int64_t i, EventKin<N>& ev, PermLds perm,
                                            bool store = true) {
  constexpr int NF = N - 2;
  const uint64_t e = C.first_event + (uint64_t)i;
  EventRng rng{(uint32_t)e, (uint32_t)(e >> 32), (uint32_t)N, C.key0, C.key1};
  const u32x4 b0 = rng.block(0);

  // colour ordering and helicities
  OrderWord<N> A;
  if (C.in_order) {
    A = 0;
#pragma unroll
    for (int t = 1; t < N; ++t) {
      // a leg index outside 1..N-1 is clamped so that malformed input never addresses
      // outside the event's arrays
      const uint32_t l = C.in_order[i * N + t];
      A |= (OrderWord<N>)(l < 1u ? 1u : (l > (uint32_t)(N - 1) ? (uint32_t)(N - 1) : l)) << (4 * (t - 1));
    }
  } else if (C.random_order) {
    A = shuffle_order<N>(rng);
  } else {
    A = identity_order<N>();
  }
  ev.leg[0] = 0;
#pragma unroll
  for (int t = 1; t < N; ++t) ev.leg[t] = nib(A, t - 1);
  ev.hel = C.in_hel ? C.in_hel[i] : (b0.v[2] & ((1u << N) - 1u));

  // parton fractions
  double sqrt_shat;
  if (C.use_pdf) {
    if (C.in_x) {
      ev.x1 = C.in_x[2 * i];
      ev.x2 = C.in_x[2 * i + 1];
    } else {
      ev.x1 = pdf_sample(u01(b0.v[0]), C.pdf);
      ev.x2 = pdf_sample(u01(b0.v[1]), C.pdf);
    }
    ev.shat = ev.x1 * ev.x2 * C.sqrt_s * C.sqrt_s;
    sqrt_shat = sqrt_fp64(ev.shat);
  } else {
    ev.x1 = ev.x2 = 1.0;
    ev.shat = C.sqrt_s * C.sqrt_s;
    sqrt_shat = C.sqrt_s;
  }

  // RAMBO over the outgoing legs: raw q, then the conformal map
  double q[NF][4];
  double Q[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int p = 0; p < NF; ++p) {
    double r[4];
    if (C.in_u) {
      const double* u = C.in_u + (i * NF + p) * 4;
      r[0] = u[0]; r[1] = u[1]; r[2] = u[2]; r[3] = u[3];
    } else {
      const u32x4 w = rng.block(1u + (uint32_t)p);
      r[0] = u01(w.v[0]); r[1] = u01(w.v[1]); r[2] = u01(w.v[2]); r[3] = u01(w.v[3]);
    }
    rambo_q(r[0], r[1], r[2], r[3], q[p]);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) perm.col[(4 * p + mu) * perm.stride] = q[p][mu];
    if (store && C.out.uniforms) {
      double* uo = C.out.uniforms + (i * NF + p) * 4;
      uo[0] = r[0]; uo[1] = r[1]; uo[2] = r[2]; uo[3] = r[3];
    }
  }
  // Q summed in position order (as the position-order form does, so that every launch form
  // gives bitwise the same momenta)
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const uint32_t j = ev.leg[t];
    const int slot = 4 * (int)(j >= 2u ? j - 2u : 0u);
    // 1 or 0 times the momentum, exactly: one multiply-add instead of two selects and an add
    const double out = j >= 2u ? 1.0 : 0.0;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) Q[mu] = __builtin_fma(out, perm.col[(slot + mu) * perm.stride], Q[mu]);
  }
  RamboMap map;
  map.init(Q, sqrt_shat);
  const double rr = 2.0 * sqrt_fp64(ev.x1 * ev.x2), irr = recip_refine(rr);
  const double ch = div_refined(ev.x1 + ev.x2, rr, irr), sh = div_refined(ev.x1 - ev.x2, rr, irr);
#pragma unroll
  for (int p = 0; p < NF; ++p) {
    double pc[4];
    map.apply(q[p], pc);
    ev.pl[p][0] = pc[0] * ch + pc[3] * sh;
    ev.pl[p][1] = pc[1];
    ev.pl[p][2] = pc[2];
    ev.pl[p][3] = pc[3] * ch + pc[0] * sh;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) perm.col[(4 * p + mu) * perm.stride] = pc[mu];
  }
  // positions: beams directly, outgoing legs from the lane's LDS column
#pragma unroll
  for (int t = 0; t < N; ++t) {
    const uint32_t j = ev.leg[t];
    const int slot = 4 * (int)(j >= 2u ? j - 2u : 0u);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) ev.pc[t][mu] = perm.col[(slot + mu) * perm.stride];
    if (j < 2u) {
      ev.pc[t][0] = 0.5 * sqrt_shat; ev.pc[t][1] = 0.0; ev.pc[t][2] = 0.0;
      ev.pc[t][3] = j == 0u ? 0.5 * sqrt_shat : -0.5 * sqrt_shat;
    }
  }
  if (!store) return;
  if (C.out.hel) C.out.hel[i] = ev.hel;
  if (C.out.order) {
#pragma unroll
    for (int t = 0; t < N; ++t) C.out.order[i * N + t] = (uint8_t)ev.leg[t];
  }
  if (C.out.x12) {
    C.out.x12[2 * i] = ev.x1;
    C.out.x12[2 * i + 1] = ev.x2;
  }
  if (C.out.momenta) {
    double* mo = C.out.momenta + i * N * 4;
    const double e1 = 0.5 * C.sqrt_s * ev.x1, e2 = 0.5 * C.sqrt_s * ev.x2;
    mo[0] = e1; mo[1] = 0.0; mo[2] = 0.0; mo[3] = e1;
    mo[4] = e2; mo[5] = 0.0; mo[6] = 0.0; mo[7] = -e2;
#pragma unroll
    for (int p = 0; p < NF; ++p) {
      mo[8 + 4 * p] = ev.pl[p][0]; mo[9 + 4 * p] = ev.pl[p][1];
      mo[10 + 4 * p] = ev.pl[p][2]; mo[11 + 4 * p] = ev.pl[p][3];
    }
  }
}

// eta = asinh(pz / pT) of a massless momentum with energy E and transverse momentum pT, as
// sign(pz) log((E + |pz|) / pT): the same function, since (|p| + |pz|)(|p| - |pz|) = pT^2
// and |p| = E.  E stands in for |p| (the momenta are massless up to rounding, so they agree
// to a few units of 2^-53), which saves the square root.  Every step is a sum of positive
// terms, a division or the logarithm, so the absolute error is a few units of 2^-53 |eta|
// (the cuts and Delta R only use eta through |eta| and differences); pT = 0 gives +-inf.
__device__ __forceinline__ double pseudorapidity(double pt, double pz, double e) {
#pragma clang fp contract(off)
  const double az = fabs(pz);
  return copysign(log_fp64((e + az) / pt), pz);
}

// Azimuth and pseudorapidity in FP32 to within kAngleErr (|eta| <= 20), to find the closest pair
// of jets: t = min / max of |y|, |x| and an odd polynomial for atan t on [0, 1] (least-squares
// fit weighted towards equal errors, 2.5e-7), then the octant; log2 of (E + |pz|) / pT.
constexpr float kAngleErr = 4e-6f;

__device__ __forceinline__ float azimuth_f32(float y, float x) {
  const float ax = fabsf(x), ay = fabsf(y);
  const float t = fminf(ax, ay) * __builtin_amdgcn_rcpf(fmaxf(ax, ay));
  const float z = t * t;
  float r = 0.0068117926f;
  r = __builtin_fmaf(r, z, -0.033604219f);
  r = __builtin_fmaf(r, z, 0.079623672f);
  r = __builtin_fmaf(r, z, -0.13233342f);
  r = __builtin_fmaf(r, z, 0.19807816f);
  r = __builtin_fmaf(r, z, -0.33317368f);
  r = __builtin_fmaf(r, z, 0.99999611f) * t;
  r = ay > ax ? 1.57079633f - r : r;
  r = x < 0.0f ? 3.14159265f - r : r;
  return copysignf(r, y);
}

// Whether FP32 decides the cut |eta| < eta_max of a jet with the pseudorapidity e: 1 it fails, -1 it
// passes, 0 within the error (left to FP64).  No cut at all (infinity, or anything beyond 1e30, which
// no pseudorapidity reaches) counts as 1e30: the difference to infinity would never decide, and
// every jet went through FP64 (1.8 us of 65 and 79 at n = 7, 8 FP32, 131072 events).
__host__ __device__ __forceinline__ int eta_side(float e, float eta_max) {
#pragma clang fp contract(off)
  eta_max = eta_max > 1e30f ? 1e30f : eta_max;
  const float d = fabsf(e) - eta_max;
  if (d >= 2.0f * kAngleErr + 1e-6f * eta_max) return 1;
  return d < -2.0f * kAngleErr - 1e-6f * eta_max ? -1 : 0;
}

// Delta R^2 of two jets; no fused multiply-adds: every form of the cuts rounds exactly as written
__device__ __forceinline__ double delta_r2(double eta_a, double phi_a, double eta_b, double phi_b) {
#pragma clang fp contract(off)
  const double pi = 3.14159265358979323846;
  double dphi = fabs(phi_a - phi_b);
  dphi = dphi > pi ? 2.0 * pi - dphi : dphi;
  const double deta = eta_a - eta_b;
  return deta * deta + dphi * dphi;
}

// Jet cuts and observables (Sec. 3, Sec. 4) on the outgoing legs (lab frame).  H_T is summed
// in position order through the lane's LDS column, as the position-order form sums it.
//
// R_min is one pair's Delta R, so from four jets on the FP64 arctangents and logarithms (about
// 160 instructions a jet) are evaluated for the closest pair only: FP32 angles rank the pairs,
// every pair within their error of the smallest is evaluated in FP64, and the minimum of those
// is bitwise the minimum over all pairs.  Nearly always that is one pair; a wave repeats while
// any lane has another.  The |eta| cut is decided in FP32 outside its error and in FP64 within.
// Angles that FP32 does not resolve (|eta| > 20, infinities, NaN) send every pair to FP64.
// Three jets have three pairs, which costs the same either way: below four all are evaluated.
template <int N>
__device__ __forceinline__ bool cuts(const GenClass& C, const EventKin<N>& ev, PermLds perm, double& ht,
                                     double& rmin) {
#pragma clang fp contract(off)
  constexpr int NF = N - 2;
  bool ok = true;
  double dr2min = 1e300;
  ht = 0.0;
  if constexpr (NF < 4) {
    double eta[NF], phi[NF];
#pragma unroll
    for (int p = 0; p < NF; ++p) {
      const double* m = ev.pl[p];
      const double pt = sqrt(m[1] * m[1] + m[2] * m[2]);
      eta[p] = pseudorapidity(pt, m[3], m[0]);
      phi[p] = atan2(m[2], m[1]);
      perm.col[(4 * p + 3) * perm.stride] = pt;
      ok = ok && (pt > C.pt_min) && (fabs(eta[p]) < C.eta_max);
    }
    static_for<0, NF>([&](auto ac) {
      constexpr int a = decltype(ac)::value;
      static_for<a + 1, NF>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
        dr2min = fmin(dr2min, delta_r2(eta[a], phi[a], eta[b], phi[b]));
      });
    });
  } else {
    constexpr int NP = NF * (NF - 1) / 2;  // pairs a < b at b (b - 1) / 2 + a
    float eta[NF], phi[NF];
    const float eta_max = (float)C.eta_max;
    uint32_t near = 0;  // jets whose |eta| cut FP32 does not decide
    bool resolved = true;
#pragma unroll
    for (int p = 0; p < NF; ++p) {
      const double* m = ev.pl[p];
      const double pt = sqrt_fp64(m[1] * m[1] + m[2] * m[2]);
      const double num = m[0] + fabs(m[3]);
      perm.col[(4 * p) * perm.stride] = m[1];
      perm.col[(4 * p + 1) * perm.stride] = m[2];
      perm.col[(4 * p + 2) * perm.stride] = copysign(num, m[3]);
      perm.col[(4 * p + 3) * perm.stride] = pt;
      const float fnum = (float)num, fpt = (float)pt;
      const bool fine = fnum < 1e30f && fpt > 1e-30f;  // in FP32's range
      const float e = 0.693147181f * __builtin_amdgcn_logf(fnum * __builtin_amdgcn_rcpf(fpt));
      eta[p] = copysignf(e, (float)m[3]);
      phi[p] = azimuth_f32((float)m[2], (float)m[1]);
      ok = ok && (pt > C.pt_min);
      const int side = fine ? eta_side(e, eta_max) : 0;
      ok = ok && side <= 0;
      near |= (side < 0 || !ok) ? 0u : 1u << p;
      resolved = resolved && fine && fabsf(e) <= 20.0f && fabsf(phi[p]) < 4.0f;
    }
    float d2[NP];
    float dmin = INFINITY;
    static_for<1, NF>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      static_for<0, b>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        float dphi = fabsf(phi[a] - phi[b]);
        dphi = fminf(dphi, 6.28318531f - dphi);
        const float deta = eta[a] - eta[b];
        const float v = __builtin_fmaf(deta, deta, dphi * dphi);
        d2[b * (b - 1) / 2 + a] = v;
        dmin = fminf(dmin, v);
      });
    });
    // an FP32 difference of angles is off by at most e = 2 kAngleErr per axis, so Delta R^2 by
    // 2 sqrt(2) e Delta R + 2 e^2 and 1e-6 of itself; twice that for the two pairs compared
    const float r = __builtin_amdgcn_sqrtf(dmin);
    float lim = dmin + (6.0f * 2.0f * kAngleErr) * r + 2e-6f * dmin + 16.0f * kAngleErr * kAngleErr;
    lim = resolved ? lim : INFINITY;
    using Mask = typename std::conditional<(NP <= 32), uint32_t, uint64_t>::type;
    Mask todo = 0;
    static_for<0, NP>([&](auto pc) {
      constexpr int p = decltype(pc)::value;
      todo |= !(d2[p] > lim) ? Mask(1) << p : Mask(0);
    });
    while (todo != 0) {
      const int p = NP <= 32 ? __builtin_ctz((uint32_t)todo) : __builtin_ctzll(todo);
      todo &= todo - 1;
      const int b = (int)(0.5f + __builtin_amdgcn_sqrtf(2.0f * (float)p + 0.26f)), a = p - b * (b - 1) / 2;
      double e2[2], f2[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const double* c = perm.col + 4 * (k == 0 ? a : b) * perm.stride;
        const double num = c[2 * perm.stride];
        e2[k] = copysign(log_fp64(fabs(num) / c[3 * perm.stride]), num);
        f2[k] = atan2(c[perm.stride], c[0]);
      }
      dr2min = fmin(dr2min, delta_r2(e2[0], f2[0], e2[1], f2[1]));
    }
    while (near != 0) {
      const int p = __builtin_ctz(near);
      near &= near - 1;
      const double* c = perm.col + 4 * p * perm.stride;
      ok = ok && fabs(log_fp64(fabs(c[2 * perm.stride]) / c[3 * perm.stride])) < C.eta_max;
    }
  }
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const uint32_t j = ev.leg[t];
    ht += j >= 2u ? perm.col[(4 * (int)(j >= 2u ? j - 2u : 0u) + 3) * perm.stride] : 0.0;
  }
  rmin = sqrt(dr2min);
  return ok && (dr2min > C.dr_min * C.dr_min);
}

// The same kinematics in recursion-position order throughout (lab momenta of all N legs),
// without the LDS permutation: used where one event spans several lanes, whose register
// budget the leg-order form's extra arrays exceed.
template <int N>
struct EventKinPos {
  double p[N][4];   // physical lab momenta, position order
  double pc[N][4];  // partonic centre-of-mass momenta (RAMBO frame), position order
  uint32_t leg[N];  // leg at each position
  uint32_t hel;
  double x1, x2, shat;
};

// (RAMBO evaluated per position: the beam positions repeat an outgoing leg's draws and are
// overwritten.)
template <int N>
__device__ __forceinline__ void build_event_positions(const GenClass& C, int64_t i, EventKinPos<N>& ev, bool store = true) {
  constexpr int NF = N - 2;
  const uint64_t e = C.first_event + (uint64_t)i;
  EventRng rng{(uint32_t)e, (uint32_t)(e >> 32), (uint32_t)N, C.key0, C.key1};
  const u32x4 b0 = rng.block(0);

  // colour ordering and helicities
  OrderWord<N> A;
  if (C.in_order) {
    A = 0;
#pragma unroll
    for (int t = 1; t < N; ++t) {
      // a leg index outside 1..N-1 is clamped so that malformed input never addresses
      // outside the event's arrays
      const uint32_t l = C.in_order[i * N + t];
      A |= (OrderWord<N>)(l < 1u ? 1u : (l > (uint32_t)(N - 1) ? (uint32_t)(N - 1) : l)) << (4 * (t - 1));
    }
  } else if (C.random_order) {
    A = shuffle_order<N>(rng);
  } else {
    A = identity_order<N>();
  }
  ev.leg[0] = 0;
#pragma unroll
  for (int t = 1; t < N; ++t) ev.leg[t] = nib(A, t - 1);
  ev.hel = C.in_hel ? C.in_hel[i] : (b0.v[2] & ((1u << N) - 1u));

  // parton fractions
  double sqrt_shat;
  if (C.use_pdf) {
    if (C.in_x) {
      ev.x1 = C.in_x[2 * i];
      ev.x2 = C.in_x[2 * i + 1];
    } else {
      ev.x1 = pdf_sample(u01(b0.v[0]), C.pdf);
      ev.x2 = pdf_sample(u01(b0.v[1]), C.pdf);
    }
    ev.shat = ev.x1 * ev.x2 * C.sqrt_s * C.sqrt_s;
    sqrt_shat = sqrt_fp64(ev.shat);
  } else {
    ev.x1 = ev.x2 = 1.0;
    ev.shat = C.sqrt_s * C.sqrt_s;
    sqrt_shat = C.sqrt_s;
  }

  // RAMBO in position order: raw q for outgoing legs, then the conformal map
  double q[N][4];
  double Q[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const uint32_t j = ev.leg[t];
    const bool out = j >= 2u;
    const uint32_t pidx = out ? j - 2u : 0u;
    double r[4];
    if (C.in_u) {
      const double* u = C.in_u + (i * NF + pidx) * 4;
      r[0] = u[0]; r[1] = u[1]; r[2] = u[2]; r[3] = u[3];
    } else {
      const u32x4 w = rng.block(1u + pidx);
      r[0] = u01(w.v[0]); r[1] = u01(w.v[1]); r[2] = u01(w.v[2]); r[3] = u01(w.v[3]);
    }
    rambo_q(r[0], r[1], r[2], r[3], q[t]);
    if (out) {
#pragma unroll
      for (int mu = 0; mu < 4; ++mu) Q[mu] += q[t][mu];
      if (store && C.out.uniforms) {
        double* uo = C.out.uniforms + (i * NF + pidx) * 4;
        uo[0] = r[0]; uo[1] = r[1]; uo[2] = r[2]; uo[3] = r[3];
      }
    }
  }
  RamboMap map;
  map.init(Q, sqrt_shat);
  const double rr = 2.0 * sqrt_fp64(ev.x1 * ev.x2), irr = recip_refine(rr);
  const double ch = div_refined(ev.x1 + ev.x2, rr, irr), sh = div_refined(ev.x1 - ev.x2, rr, irr);
  const double e1 = 0.5 * C.sqrt_s * ev.x1, e2 = 0.5 * C.sqrt_s * ev.x2;
#pragma unroll
  for (int t = 0; t < N; ++t) {
    const uint32_t j = ev.leg[t];
    double pc[4];
    map.apply(q[t], pc);  // harmless for beam positions, overwritten below
    double pl[4] = {pc[0] * ch + pc[3] * sh, pc[1], pc[2], pc[3] * ch + pc[0] * sh};
    if (j == 0u) {
      pl[0] = e1; pl[1] = 0.0; pl[2] = 0.0; pl[3] = e1;
      pc[0] = 0.5 * sqrt_shat; pc[1] = 0.0; pc[2] = 0.0; pc[3] = 0.5 * sqrt_shat;
    } else if (j == 1u) {
      pl[0] = e2; pl[1] = 0.0; pl[2] = 0.0; pl[3] = -e2;
      pc[0] = 0.5 * sqrt_shat; pc[1] = 0.0; pc[2] = 0.0; pc[3] = -0.5 * sqrt_shat;
    }
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      ev.p[t][mu] = pl[mu];
      ev.pc[t][mu] = pc[mu];
    }
  }
  if (!store) return;
  if (C.out.hel) C.out.hel[i] = ev.hel;
  if (C.out.order) {
#pragma unroll
    for (int t = 0; t < N; ++t) C.out.order[i * N + t] = (uint8_t)ev.leg[t];
  }
  if (C.out.x12) {
    C.out.x12[2 * i] = ev.x1;
    C.out.x12[2 * i + 1] = ev.x2;
  }
  if (C.out.momenta) {
#pragma unroll
    for (int t = 0; t < N; ++t) {
      double* mo = C.out.momenta + (i * N + ev.leg[t]) * 4;
      mo[0] = ev.p[t][0]; mo[1] = ev.p[t][1]; mo[2] = ev.p[t][2]; mo[3] = ev.p[t][3];
    }
  }
}

// cuts() on position-ordered lab momenta (the beam positions masked).
template <int N>
__device__ __forceinline__ bool cuts_positions(const GenClass& C, const EventKinPos<N>& ev, double& ht, double& rmin) {
#pragma clang fp contract(off)
  double pt[N], eta[N], phi[N];
  bool ok = true;
  ht = 0.0;
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double* p = ev.p[t];
    pt[t] = sqrt(p[1] * p[1] + p[2] * p[2]);
    eta[t] = pseudorapidity(pt[t], p[3], p[0]);
    phi[t] = atan2(p[2], p[1]);
    const bool out = ev.leg[t] >= 2u;
    if (out) {
      ht += pt[t];
      ok = ok && (pt[t] > C.pt_min) && (fabs(eta[t]) < C.eta_max);
    }
  }
  double dr2min = 1e300;
  const double pi = 3.14159265358979323846;
  static_for<1, N>([&](auto tc) {
    constexpr int t = decltype(tc)::value;
    static_for<t + 1, N>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      double dphi = fabs(phi[t] - phi[u]);
      dphi = dphi > pi ? 2.0 * pi - dphi : dphi;
      const double deta = eta[t] - eta[u];
      const double d2 = deta * deta + dphi * dphi;
      const bool both = (ev.leg[t] >= 2u) && (ev.leg[u] >= 2u);
      dr2min = both ? fmin(dr2min, d2) : dr2min;
    });
  });
  rmin = sqrt(dr2min);
  return ok && (dr2min > C.dr_min * C.dr_min);
}

// |A(sigma;h)|^2 from position-ordered physical momenta.  Momenta are scaled by the power
// of two 2^-ex nearest below half their summed energy (exact in binary floating point),
// and |A|^2(k) = 2^(2 ex (4-N)) |A|^2(2^-ex k).
template <int N, typename T>
struct UseLdsK {
  static constexpr bool value = lds_span_table(N, std::is_same<T, float>::value ? 32 : 64);
};

// The LDS span table of one workgroup (only instantiated where UseLdsK holds): momenta of every
// span but the full one, propagators of the spans of 2..N-2 legs.
template <int N>
struct LdsTable {
  float4 k[(Spans<N - 1>::count - 1) * kLdsLanes];
  float p[(Spans<N - 1>::count - N) * kLdsLanes];
};

// |A|^2 past an optimisation barrier: without it the compiler sinks parts of the recursion below
// the branches of the outputs that follow, where its live values spill (FP64 n = 8: 3 KB of
// scratch per lane).
__device__ __forceinline__ double rec_done(double a2) {
  opaque(a2);
  return a2;
}

// The LDS of a one-lane recursion's workgroup (kLdsLanes lanes): the FP32 span table, or the FP64
// leg momenta and span scalars.
template <int N, typename T>
using RecLds = typename std::conditional<std::is_same<T, float>::value, LdsTable<N>, Fp64Lds<N - 1, kLdsLanes>>::type;

template <int N, typename T, bool LDS>
__device__ __forceinline__ double ordered_amp2(const double (&p)[N][4], const uint32_t (&leg)[N], uint32_t hel,
                                               RecLds<N, T>* tab) {
  double esum = 0.0;
#pragma unroll
  for (int t = 0; t < N; ++t) esum += fabs(p[t][0]);
  const int ex = ilogb(0.5 * esum);
  const double sc = ldexp(1.0, -ex);
  double k[N - 1][4];
  cv4<T> src[N - 1];
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double sg = leg[t] < 2u ? -sc : sc;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) k[t - 1][mu] = sg * p[t][mu];
    src[t - 1] = polarisation<T>(p[t], (hel >> leg[t]) & 1u);
  }
  const cv4<T> e0 = polarisation<T>(p[0], (hel >> leg[0]) & 1u);
  double mr, mi;
  if constexpr (LDS && std::is_same<T, double>::value) {
    __syncthreads();  // as below
    const Fp64Span<N - 1, kLdsLanes> ks{tab->leg + threadIdx.x, tab->sc + threadIdx.x};
#pragma unroll
    for (int t = 0; t < N - 1; ++t) ks.put_leg(t, k[t]);
    bg_amplitude_d<N - 1, kLdsLanes>(ks, src, e0, mr, mi);
  } else if constexpr (LDS) {
    // the generation kernel carries its momentum permutation (doubles) in this memory: the
    // barrier keeps the compiler from moving the table fill above those accesses (the
    // workgroup is one wave, so it costs nothing else)
    __syncthreads();
    SpanKLds<N - 1, kLdsLanes> ks{tab->k + threadIdx.x, tab->p + threadIdx.x};
    ks.fill(k);
    bg_amplitude<N - 1, T>(ks, src, e0, mr, mi);
  } else {
    SpanKLegs<N - 1, T> ks{k};
    bg_amplitude<N - 1, T>(ks, src, e0, mr, mi);
  }
  return rec_done(ldexp(__builtin_fma(mr, mr, mi * mi), 2 * ex * (4 - N) - (N - 2)));
}

// Angles of the real polarisations of an event (random_polarisation): leg k takes word k % 4
// of Philox block n_blocks + k / 4 (after the draws of the helicity mode), psi = 2 pi u;
// returns cos psi, sin psi per leg, evaluated in FP64.
template <int N>
__device__ __forceinline__ void polarisation_angles(const GenClass& C, int64_t i, double (&cs)[N][2]) {
  const uint64_t e = C.first_event + (uint64_t)i;
  const EventRng rng{(uint32_t)e, (uint32_t)(e >> 32), (uint32_t)N, C.key0, C.key1};
  constexpr uint32_t b0 = 1u + (N - 2) + (N - 2 + 3) / 4;
  u32x4 w{};
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if ((k & 3) == 0) w = rng.block(b0 + (uint32_t)(k / 4));
    sincospi_fp64(2.0 * u01(w.v[k & 3]), &cs[k][1], &cs[k][0]);
  }
}

// |A(sigma; eps_psi)|^2 with real polarisations (cs: cos, sin of each leg's angle), as
// ordered_amp2.
template <int N, typename T, bool LDS>
__device__ __forceinline__ double ordered_amp2_real(const double (&p)[N][4], const uint32_t (&leg)[N],
                                                    const double (&cs)[N][2], RecLds<N, T>* tab) {
  double esum = 0.0;
#pragma unroll
  for (int t = 0; t < N; ++t) esum += fabs(p[t][0]);
  const int ex = ilogb(0.5 * esum);
  const double sc = ldexp(1.0, -ex);
  double k[N - 1][4];
  rv4<T> src[N - 1];
  // the angle of the leg at each position, selected without dynamic register indexing
  auto angle = [&](uint32_t l, T& c, T& s) {
    double cd = cs[0][0], sd = cs[0][1];
#pragma unroll
    for (int q = 1; q < N; ++q) {
      cd = l == (uint32_t)q ? cs[q][0] : cd;
      sd = l == (uint32_t)q ? cs[q][1] : sd;
    }
    c = T(cd);
    s = T(sd);
  };
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double sg = leg[t] < 2u ? -sc : sc;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) k[t - 1][mu] = sg * p[t][mu];
    T c, s;
    angle(leg[t], c, s);
    src[t - 1] = real_polarisation<T>(p[t], c, s);
  }
  T c0, s0;
  angle(leg[0], c0, s0);
  const rv4<T> e0 = real_polarisation<T>(p[0], c0, s0);
  double m;
  if constexpr (LDS) {
    __syncthreads();
    SpanKLds<N - 1, kLdsLanes> ks{tab->k + threadIdx.x, tab->p + threadIdx.x};
    ks.fill(k);
    m = bg_amplitude_r<N - 1, T>(ks, src, e0);
  } else {
    SpanKLegs<N - 1, T> ks{k};
    m = bg_amplitude_r<N - 1, T>(ks, src, e0);
  }
  return rec_done(ldexp(m * m, 2 * ex * (4 - N) - (N - 2)));
}

// The same with the event spread over the G lanes of a group (FP32; FP64 groups:
// ordered_amp2_p, ordered_amp2_q); g is this lane's place in it.  The span momenta and propagators
// come from the workgroup's table lds (SpanKGroupLds).
template <int N, typename T, int G>
__device__ __forceinline__ double ordered_amp2_g(const double (&p)[N][4], const uint32_t (&leg)[N], uint32_t hel,
                                                 int g, unsigned char* lds) {
  constexpr int C = 4 / G;
  double esum = 0.0;
#pragma unroll
  for (int t = 0; t < N; ++t) esum += fabs(p[t][0]);
  const int ex = ilogb(0.5 * esum);
  const double sc = ldexp(1.0, -ex);
  const LaneShare<G, T> ls(g);
  const LaneShare<G, double> lsd(g);
  double k[N - 1][C];  // covariant, this lane's components
  cvl<T, C> src[N - 1], e0;
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double sg = leg[t] < 2u ? -sc : sc;
#pragma unroll
    for (int c = 0; c < C; ++c) k[t - 1][c] = lsd.sg[c] * (sg * lsd.pick(p[t], c));
    const cv4<T> e = polarisation<T>(p[t], (hel >> leg[t]) & 1u);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      src[t - 1].re[c] = ls.pick(e.re, c);
      src[t - 1].im[c] = ls.pick(e.im, c);
    }
  }
  {
    const cv4<T> e = polarisation<T>(p[0], (hel >> leg[0]) & 1u);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      e0.re[c] = ls.pick(e.re, c);
      e0.im[c] = ls.pick(e.im, c);
    }
  }
  double mr, mi;
  const SpanKGroupLds<N - 1, G, T> ks(k, lsd.sg, lds, (int)threadIdx.x, (int)blockDim.x);
  bg_amplitude_g<N - 1, G, T>(ls, ks, src, e0, mr, mi);
  return rec_done(ldexp(__builtin_fma(mr, mr, mi * mi), 2 * ex * (4 - N) - (N - 2)));
}

// FP64 on a lane pair (PairSpan); lds: the workgroup's pair_lds_bytes<N - 1>() per lane.
template <int N>
__device__ __forceinline__ double ordered_amp2_p(const double (&p)[N][4], const uint32_t (&leg)[N], uint32_t hel,
                                                 unsigned char* lds) {
  const PairSpan<N - 1> ks(lds, (int)threadIdx.x, (int)blockDim.x);
  double esum = 0.0;
#pragma unroll
  for (int t = 0; t < N; ++t) esum += fabs(p[t][0]);
  const int ex = ilogb(0.5 * esum);
  const double sc = ldexp(1.0, -ex);
  cvp src[N - 1], e0;
  auto share = [&](const cv4<double>& e) {
    cvp s;
    s.re[0] = ks.g ? e.re[3] : 0.0;
    s.im[0] = 0.0;
    s.re[1] = ks.g ? e.re[2] : e.re[1];
    s.im[1] = ks.g ? e.im[2] : e.im[1];
    return s;
  };
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double sg = leg[t] < 2u ? -sc : sc;
    const double first = ks.g ? p[t][3] : p[t][0], second = ks.g ? p[t][2] : p[t][1];
    ks.leg[(t - 1) * ks.lanes] = make_double2(ks.sg * (sg * first), -(sg * second));
    src[t - 1] = share(polarisation<double>(p[t], (hel >> leg[t]) & 1u));
  }
  e0 = share(polarisation<double>(p[0], (hel >> leg[0]) & 1u));
  double mr, mi;
  bg_amplitude_p<N - 1>(ks, src, e0, mr, mi);
  return rec_done(ldexp(__builtin_fma(mr, mr, mi * mi), 2 * ex * (4 - N) - (N - 2)));
}

// FP64 on four lanes (QuadSpan: lane 16 c + e of the wave holds component c of event e); lds: the
// wave's quad_lds_bytes<N - 1>().  Called by every lane of the wave.
template <int N>
__device__ __forceinline__ double ordered_amp2_q(const double (&p)[N][4], const uint32_t (&leg)[N], uint32_t hel,
                                                 unsigned char* lds) {
  const QuadSpan<N - 1> ks(lds, (int)(threadIdx.x & 63u));
  double esum = 0.0;
#pragma unroll
  for (int t = 0; t < N; ++t) esum += fabs(p[t][0]);
  const int ex = ilogb(0.5 * esum);
  const double sc = ldexp(1.0, -ex);
  cvq src[N - 1], e0;
  auto share = [&](cv4<double> e) {
    // (past a barrier: the compiler would branch on the component instead of selecting)
#pragma unroll
    for (int mu = 1; mu < 4; ++mu) opaque(e.re[mu]);
    opaque(e.im[1]);
    opaque(e.im[2]);
    return cvq{ks.c == 1 ? e.re[1] : (ks.c == 2 ? e.re[2] : (ks.c == 3 ? e.re[3] : 0.0)),
               ks.c == 1 ? e.im[1] : (ks.c == 2 ? e.im[2] : 0.0)};
  };
#pragma unroll
  for (int t = 1; t < N; ++t) {
    const double sg = leg[t] < 2u ? -sc : sc;
    const double mine = ks.c < 2 ? (ks.c == 0 ? p[t][0] : p[t][1]) : (ks.c == 2 ? p[t][2] : p[t][3]);
    ks.leg[(t - 1) * 64] = ks.sg * (sg * mine);
    src[t - 1] = share(polarisation<double>(p[t], (hel >> leg[t]) & 1u));
  }
  e0 = share(polarisation<double>(p[0], (hel >> leg[0]) & 1u));
  double mr, mi;
  bg_amplitude_q<N - 1>(ks, src, e0, mr, mi);
  return rec_done(ldexp(__builtin_fma(mr, mr, mi * mi), 2 * ex * (4 - N) - (N - 2)));
}

// Compensated (sum w, sum w^2) of a workgroup of up to 256 lanes, in a fixed tree order;
// thread 0 stores (s, c, s2, c2) to dst.  A wave whose lanes all hold zeros (every event failed
// the cuts: 80% of the waves of 64 events at n = 8 and sqrt(S) = 14 TeV) has zero sums and
// skips its six exchange steps, a chain of some 1500 cycles that one wave per SIMD cannot hide;
// a workgroup of one wave needs no exchange through LDS.
__device__ __forceinline__ void block_reduce_store(CSum w, CSum w2, double* dst) {
  if (__any(w.s != 0.0 || w.c != 0.0 || w2.s != 0.0 || w2.c != 0.0)) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      CSum ow{__shfl_down(w.s, off), __shfl_down(w.c, off)};
      CSum ow2{__shfl_down(w2.s, off), __shfl_down(w2.c, off)};
      w = cs_add(w, ow);
      w2 = cs_add(w2, ow2);
    }
  }
  if (blockDim.x > 64) {
    __shared__ double red[4][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
      red[wave][0] = w.s; red[wave][1] = w.c; red[wave][2] = w2.s; red[wave][3] = w2.c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      w = CSum{red[0][0], red[0][1]};
      w2 = CSum{red[0][2], red[0][3]};
      const int nw = (int)(blockDim.x >> 6);
      for (int v = 1; v < nw; ++v) {
        w = cs_add(w, CSum{red[v][0], red[v][1]});
        w2 = cs_add(w2, CSum{red[v][2], red[v][3]});
      }
    }
  }
  if (threadIdx.x == 0) {
    dst[0] = w.s; dst[1] = w.c; dst[2] = w2.s; dst[3] = w2.c;
  }
}

// The weight of Eq. 3.8 from |A|^2 (w = 0 exactly when the event fails the cuts, never
// 0 times a product), and the per-event outputs of |A|^2, the weight, the cut flag and the
// log integrand weight; returns w.  Shared by every generation kernel, so that each
// output rounds identically whichever kernel evaluates the event.
// Dynamic scale mu = H_T: alpha_s(mu)^(n-2) f(x1, mu) f(x2, mu) over the factors at mu0 that
// wconst and the sampling density hold (exactly 1 with a fixed scale).
template <int N>
__device__ __forceinline__ double scale_ratio(const GenClass& C, double ht, double x1, double x2) {
#pragma clang fp contract(off)
  if (!C.dynamic_scale) return 1.0;
  const double lmu = log(ht);
  double lr = double(N - 2) * (log(grid_alpha(C.grid, lmu)) - C.log_alpha0);
  if (C.use_pdf) {
    const double l1 = log(x1), l2 = log(x2), m1 = log1p(-x1), m2 = log1p(-x2);
    lr += (grid_lnf(C.grid, lmu, l1 - m1) - (C.pdf.a * l1 + double(C.pdf.b) * m1)) +
          (grid_lnf(C.grid, lmu, l2 - m2) - (C.pdf.a * l2 + double(C.pdf.b) * m2));
  }
  return exp(lr);
}

// r: scale_ratio of the event.
template <int N>
__device__ __forceinline__ double finish_event(const GenClass& C, int64_t i, bool pass, double a2, double shat,
                                               double x1, double x2, double r) {
#pragma clang fp contract(off)
  double sp = 1.0;
#pragma unroll
  for (int k = 0; k < (N > 5 ? N - 5 : 5 - N); ++k) sp *= shat;
  if (N < 5) sp = 1.0 / sp;
  const double w = pass ? C.wconst * sp * a2 * r : 0.0;
  if (C.out.weight) C.out.weight[i] = w;
  if (C.out.amp2) C.out.amp2[i] = a2;
  if (C.out.pass) C.out.pass[i] = pass ? 1 : 0;
  if (C.out.logw) {
    double lw = log(a2) + double(N - 5) * log(shat) + C.log_const;
    if (C.use_pdf) lw += C.pdf.a * (log(x1) + log(x2)) + double(C.pdf.b) * (log1p(-x1) + log1p(-x2));
    if (C.dynamic_scale) lw += log(r);
    C.out.logw[i] = a2 > 0.0 ? lw : -INFINITY;
  }
  return w;
}

// One event: draws -> kinematics -> cuts -> |A|^2 -> weight; writes outputs; returns w.
// With G > 1 lanes per event every lane of the group evaluates the kinematics (the same
// values), the recursion is shared, and lane g = 0 writes the outputs and returns w
// (the others return 0).
// With LDS (one lane) the recursion uses the workgroup's table tab, which may lie over the memory
// of perm: the kinematics are done with it by then.  With G > 1, tab holds SpanKGroupLds.
template <int N, typename T, int G = 1, int POL = 0, bool LDS = false>
__device__ __forceinline__ double generate_one(const GenClass& C, int64_t i, PermLds perm, int g = 0,
                                               RecLds<N, T>* tab = nullptr) {
  static_assert(POL == 0 || G == 1, "real polarisations run one lane per event");
  using Kin = typename std::conditional<G == 1, EventKin<N>, EventKinPos<N>>::type;
  Kin ev;
  double ht, rmin;
  bool pass;
  if constexpr (G == 1) {
    build_event<N>(C, i, ev, perm, g == 0);
    pass = cuts<N>(C, ev, perm, ht, rmin);
  } else {
    (void)perm;
    build_event_positions<N>(C, i, ev, g == 0);
    pass = cuts_positions<N>(C, ev, ht, rmin);
  }
  const double r = scale_ratio<N>(C, ht, ev.x1, ev.x2);
  if (C.out.obs && g == 0) {
    C.out.obs[2 * i] = ht;
    C.out.obs[2 * i + 1] = rmin;
  }
  // |A|^2 is Lorentz invariant: evaluated in the partonic centre-of-mass frame
  double a2;
  if constexpr (POL == 1) {
    double cs[N][2];
    polarisation_angles<N>(C, i, cs);
    a2 = ordered_amp2_real<N, T, LDS>(ev.pc, ev.leg, cs, tab);
  } else if constexpr (G == 1) {
    a2 = ordered_amp2<N, T, LDS>(ev.pc, ev.leg, ev.hel, tab);
  } else {
    a2 = ordered_amp2_g<N, T, G>(ev.pc, ev.leg, ev.hel, g, reinterpret_cast<unsigned char*>(tab));
  }
  if (g != 0) return 0.0;
  return finish_event<N>(C, i, pass, a2, ev.shat, ev.x1, ev.x2, r);
}

// Waves per SIMD the compiler may leave room for in the one-lane recursion kernels.  A limit of
// one pads the register allocation beyond 256, so that a second wave never fits, and is kept
// only where the recursion needs that many: below, several waves hide the latency of the loads
// and of the FP64 chains (n = 4 FP32 recursion kernel, 2^22 events: 242 us at one wave, 170 us
// at seven).  FP64 n = 6 fits 256 registers when told to (264 otherwise).
template <int N, typename T, int POL>
constexpr int rec_waves() {
  constexpr int words = (Spans<N - 1>::count * (POL == 0 ? 8 : 4) + 2 * N) * (int)(sizeof(T) / 4);
  return words > (sizeof(T) == 8 && UseLdsK<N, T>::value && POL == 0 ? 270 : 210) ? 1 : 8;
}
template <int N, typename T, int POL>
constexpr int rec_waves_min() { return sizeof(T) == 8 && POL == 0 && N == 6 ? 2 : 1; }

// Single-class generation in one kernel, the classes with n <= 6: one event per lane, the
// kinematics' momentum permutation and the recursion's table in the same LDS, one compensated
// partial per 64 events.  Launch: kLdsLanes threads; partials may be NULL.
template <int N, typename T, int POL>
__global__ __launch_bounds__(kLdsLanes)
    __attribute__((amdgpu_waves_per_eu(rec_waves_min<N, T, POL>(), rec_waves<N, T, POL>()))) void k_generate_lds(
        GenClass C, double* partials) {
  constexpr unsigned kTab = sizeof(RecLds<N, T>), kPerm = perm_lds_bytes(N, kLdsLanes);
  __shared__ __align__(16) unsigned char lds[kTab > kPerm ? kTab : kPerm];
  const int64_t i = (int64_t)blockIdx.x * kLdsLanes + threadIdx.x;
  double w = 0.0;
  if (i < C.count)
    w = generate_one<N, T, 1, POL, true>(C, i, PermLds{reinterpret_cast<double*>(lds) + threadIdx.x, kLdsLanes}, 0,
                                         reinterpret_cast<RecLds<N, T>*>(lds));
  if (partials) block_reduce_store(CSum{w, 0.0}, CSum{w * w, 0.0}, partials + 4 * (int64_t)blockIdx.x);
}

// Single-class generation in one kernel without the table (FP32 n = 9 with one lane, real
// polarisations beyond FP32 n = 8 and in FP64): one event per lane, one compensated partial per
// workgroup.  Launch: blockDim.x in {64, 128, 192, 256} with perm_lds_bytes(N, blockDim.x) bytes of
// dynamic LDS; partials may be NULL.
template <int N, typename T, int POL = 0>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, rec_waves<N, T, POL>()))) void k_generate(
    GenClass C, double* partials) {
  static_assert(POL == 1 || !UseLdsK<N, T>::value, "the table classes have their own kernels");
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double w = 0.0;
  if (i < C.count) w = generate_one<N, T, 1, POL>(C, i, dyn_perm());
  if (partials) block_reduce_store(CSum{w, 0.0}, CSum{w * w, 0.0}, partials + 4 * (int64_t)blockIdx.x);
}

// |A|^2 from given momenta (bg_amp2): momenta [count][N][4] physical, gathered in colour order.
template <int N, typename T>
__global__ __launch_bounds__((UseLdsK<N, T>::value ? kLdsLanes : 256))
    __attribute__((amdgpu_waves_per_eu(rec_waves_min<N, T, 0>(), rec_waves<N, T, 0>()))) void k_amp2(
        int64_t count, const double* __restrict__ mom, const uint32_t* __restrict__ hel,
        const uint8_t* __restrict__ order, double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  double p[N][4];
  uint32_t leg[N];
#pragma unroll
  for (int t = 0; t < N; ++t) {
    const uint32_t l = order[i * N + t];
    leg[t] = l < (uint32_t)N ? l : (uint32_t)(N - 1);  // malformed input stays in bounds
    const double* q = mom + (i * N + leg[t]) * 4;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) p[t][mu] = q[mu];
  }
  if constexpr (UseLdsK<N, T>::value) {
    __shared__ RecLds<N, T> tab;
    out[i] = ordered_amp2<N, T, true>(p, leg, hel[i], &tab);
  } else {
    out[i] = ordered_amp2<N, T, false>(p, leg, hel[i], nullptr);
  }
}

// Dynamic LDS of the grouped kernels for workgroups of `block` lanes: the FP32 span-momentum
// table, or the FP64 lane pair's legs and scalars
template <int N, typename T, int G>
constexpr int grouped_lds_bytes(int block) {
  return sizeof(T) == 4 ? SpanKGroupLds<N - 1, G, T>::kBytes * block
                        : (G == 2 ? pair_lds_bytes<N - 1>() * block : quad_lds_bytes<N - 1>() * (block / 64));
}

// Waves per SIMD of the grouped kernels.  Four-lane FP64 runs two, which cover the latency of
// the matrix sums and the LDS: at n = 12 that means 480 B of scratch per lane (bg_amp2 520), but one wave
// without scratch is slower (2^18 events: n = 11 731 -> 598 us, n = 12 1000 -> 868 us; n = 10 fits).
// Elsewhere the currents take more than half the registers.
template <typename T, int G>
constexpr int group_waves() { return sizeof(T) == 8 && G == 4 ? 2 : 1; }

// The event of a lane within its workgroup's blockDim.x / G, and the lane's place in its group:
// adjacent lanes, or the matrix cores' columns for FP64 on four lanes.
template <typename T, int G>
__device__ __forceinline__ void group_place(int& event, int& g) {
  if constexpr (G == 4 && sizeof(T) == 8) {
    event = (int)(threadIdx.x >> 6) * 16 + (int)(threadIdx.x & 15u);
    g = (int)(threadIdx.x >> 4) & 3;
  } else {
    event = (int)threadIdx.x / G;
    g = (int)threadIdx.x % G;
  }
}

// |A|^2 of an event on the G lanes of a group; gdyn: the workgroup's dynamic LDS.
template <int N, typename T, int G>
__device__ __forceinline__ double grouped_amp2(const double (&p)[N][4], const uint32_t (&leg)[N], uint32_t hel, int g,
                                               unsigned char* gdyn) {
  if constexpr (G == 2 && sizeof(T) == 8)
    return ordered_amp2_p<N>(p, leg, hel, gdyn);
  else if constexpr (G == 4 && sizeof(T) == 8)
    return ordered_amp2_q<N>(p, leg, hel, gdyn + (threadIdx.x >> 6) * quad_lds_bytes<N - 1>());
  else
    return ordered_amp2_g<N, T, G>(p, leg, hel, g, gdyn);
}

// bg_amp2 with G lanes per event.  Dynamic LDS: grouped_lds_bytes.
template <int N, typename T, int G>
__global__ __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(group_waves<T, G>(), group_waves<T, G>()))) void k_amp2_g(
    int64_t count, const double* __restrict__ mom, const uint32_t* __restrict__ hel, const uint8_t* __restrict__ order,
    double* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char gdyn[];
  int event, g;
  group_place<T, G>(event, g);
  // every lane runs the recursion (QuadSpan); those past the end repeat the last event
  const int64_t ii = (int64_t)blockIdx.x * (blockDim.x / G) + event;
  const int64_t i = ii < count ? ii : count - 1;
  double p[N][4];
  uint32_t leg[N];
#pragma unroll
  for (int t = 0; t < N; ++t) {
    const uint32_t l = order[i * N + t];
    leg[t] = l < (uint32_t)N ? l : (uint32_t)(N - 1);  // malformed input stays in bounds
    const double* q = mom + (i * N + leg[t]) * 4;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) p[t][mu] = q[mu];
  }
  const double a2 = grouped_amp2<N, T, G>(p, leg, hel[i], g, gdyn);
  if (g == 0 && ii < count) out[i] = a2;
}

}  // namespace bgk
