// Generation of a class as two kernels (n = 7, 8 one event per lane; two or four lanes per event;
// the staged classes of the persistent multi-class launch): k_kin evaluates the
// kinematics (draws, parton fractions, RAMBO, boost, cuts) at several waves per SIMD, which
// hides the latency of its long FP64 chains, and hands each event's centre-of-mass momenta,
// s_hat, x1, x2, helicity word, cut flag and leg positions to k_rec through a staging
// buffer; k_rec evaluates |A|^2 at the recursion's register budget (one wave per SIMD), the
// weight and one compensated partial per 64 events.  The per-event bodies (kin_one, rec_one)
// are also the table classes' part of the persistent multi-class kernel, so an event gives
// bitwise the same values in either launch.
#pragma once

#include <algorithm>

#include "bg_kernels.hpp"
#include "bg_launch.hpp"

namespace bgk {

// Staging layout: events in tiles of 64 (one wave), each tile holding its words one after
// another, word w of event j at buf[((j / 64) * kWords + w) * 64 + j % 64], so that a wave
// reads one contiguous block.  Words: the centre-of-mass momenta of recursion positions
// 1..N-1 (position t, component mu at 4 (t - 1) + mu; position 0 is always the beam leg 0,
// which follows from s_hat), s_hat, the packed word (EventWord); then, written and read only
// when they are used, x1, x2 (with the log w output) and the weight factor of the dynamic scale
// (scale_ratio).
template <int N>
struct SplitLayout {
  static constexpr int kMom = 0, kShat = 4 * (N - 1), kMeta = kShat + 1, kX1 = kShat + 2, kX2 = kShat + 3,
                       kR = kShat + 4, kWords = kShat + 5;
  static constexpr int kAlways = kMeta + 1;  // words that every event stages
  static_assert(kWords == split_words(N), "staging words");
  __device__ static int64_t at(int64_t j, int w) { return ((j >> 6) * kWords + w) * 64 + (j & 63); }
};

// The helicity bits (0..11), the cut flag (12) and the legs at positions 1..N-1 (four bits each
// from bit 16) of one event in a word.
template <int N>
struct EventWord {
  uint64_t v;
  __device__ __forceinline__ static EventWord pack(uint32_t hel, bool pass, const uint32_t (&leg)[N]) {
    uint64_t w = (hel & 0xFFFu) | (pass ? 1u << 12 : 0u);
#pragma unroll
    for (int t = 1; t < N; ++t) w |= (uint64_t)(leg[t] & 15u) << (12 + 4 * t);
    return EventWord{w};
  }
  __device__ __forceinline__ uint32_t hel() const { return (uint32_t)v & 0xFFFu; }
  __device__ __forceinline__ bool pass() const { return (((uint32_t)v >> 12) & 1u) != 0; }
  __device__ __forceinline__ void legs(uint32_t (&leg)[N]) const {
    leg[0] = 0;
#pragma unroll
    for (int t = 1; t < N; ++t) leg[t] = (uint32_t)(v >> (12 + 4 * t)) & 15u;
  }
};

// The events that pass the cuts, where nothing of the others is asked for but their weight, which is
// zero (no |A|^2, no log w; the rule: pass_listed).  k_kin leaves one mask per 64 events, k_pass_list
// turns the masks into the list of the passing events' slots in event order, k_rec / k_rec_g run
// on that list, leaving each weight in its event's slot, and k_sum_weights forms the partials from
// the slots in the recursion kernels' launch shapes: every value and the totals are bitwise those
// of the route over every event, which is also what runs when all of them pass.  List and weights
// lie in the words of the slots that only the log w output uses.
struct PassList {
  const uint64_t* count;  // passing events; NULL: no list, every event
  double* stage;
};

// Slot of the list's entry l
template <int N>
__device__ __forceinline__ int64_t pass_slot(const double* __restrict__ buf, int64_t l) {
  return __double_as_longlong(buf[SplitLayout<N>::at(l, SplitLayout<N>::kX1)]);
}

// Kinematics of event i (staging slot j): writes the cut flag and observables and stages
// the event.  perm: the lane's LDS column (perm_lds_bytes).  Bound by VALU issue (92% of the
// SIMD's slots at n = 8 with three waves), so what counts is instructions: 3638 -> 2880 per wave
// at n = 8 with the closest pair's angles alone in FP64 (cuts), Horner coefficients in scalar
// registers (coef), divisions and roots without range scaling and three-way exclusive ors;
// 461 -> 400 us per 2^22 events at n = 8, 234 -> 199 us at n = 4.
template <int N>
__device__ __forceinline__ void kin_one(const GenClass& C, int64_t i, int64_t j, double* __restrict__ buf,
                                        PermLds perm, uint64_t* passed = nullptr) {
  using L = SplitLayout<N>;
  EventKin<N> ev;
  double ht, rmin;
  build_event<N>(C, i, ev, perm, true);
  // staged before the cuts, which then have the registers
#pragma unroll
  for (int t = 1; t < N; ++t)
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) buf[L::at(j, L::kMom + 4 * (t - 1) + mu)] = ev.pc[t][mu];
  buf[L::at(j, L::kShat)] = ev.shat;
  if (C.out.logw) {
    buf[L::at(j, L::kX1)] = ev.x1;
    buf[L::at(j, L::kX2)] = ev.x2;
  }
  const bool pass = cuts<N>(C, ev, perm, ht, rmin);
  if (C.out.pass) C.out.pass[i] = pass ? 1 : 0;
  if (C.out.obs) {
    C.out.obs[2 * i] = ht;
    C.out.obs[2 * i + 1] = rmin;
  }
  if (C.dynamic_scale) buf[L::at(j, L::kR)] = scale_ratio<N>(C, ht, ev.x1, ev.x2);
  buf[L::at(j, L::kMeta)] = __longlong_as_double((long long)EventWord<N>::pack(ev.hel, pass, ev.leg).v);
  if (passed) {
    const uint64_t m = __ballot(pass);
    if ((threadIdx.x & 63u) == 0) passed[j >> 6] = m;
    if (!pass) {
      if (C.out.weight) C.out.weight[i] = 0.0;
      buf[L::at(j, L::kX2)] = 0.0;
    }
  }
}

// One event's staged words in registers.
template <int N>
struct Staged {
  double pc[N - 1][4];  // positions 1..N-1
  double shat;
  EventWord<N> word;
};

template <int N>
__device__ __forceinline__ void load_staged(const double* __restrict__ buf, int64_t j, Staged<N>& s) {
  using L = SplitLayout<N>;
#pragma unroll
  for (int t = 1; t < N; ++t)
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) s.pc[t - 1][mu] = buf[L::at(j, L::kMom + 4 * (t - 1) + mu)];
  s.shat = buf[L::at(j, L::kShat)];
  s.word.v = (uint64_t)__double_as_longlong(buf[L::at(j, L::kMeta)]);
}

// The weight and outputs of a staged event; its optional words are read here, where used.
template <int N>
__device__ __forceinline__ double finish_staged(const GenClass& C, int64_t i, int64_t j, const double* __restrict__ buf,
                                                bool pass, double a2, double shat) {
  using L = SplitLayout<N>;
  double x1 = 1.0, x2 = 1.0, r = 1.0;
  if (C.out.logw) {
    x1 = buf[L::at(j, L::kX1)];
    x2 = buf[L::at(j, L::kX2)];
  }
  if (C.dynamic_scale) r = buf[L::at(j, L::kR)];
  return finish_event<N>(C, i, pass, a2, shat, x1, x2, r);
}

// |A|^2, weight and outputs of event i from its staged words (one lane per event, the span
// table in tab); returns w.
template <int N, typename T, int POL>
__device__ __forceinline__ double rec_staged(const GenClass& C, int64_t i, int64_t j, const double* __restrict__ buf,
                                             const Staged<N>& s, RecLds<N, T>* tab) {
  double pc[N][4];
  // position 0: the beam leg 0, as build_event forms it
  const double hb = 0.5 * (C.use_pdf ? sqrt(s.shat) : C.sqrt_s);
  pc[0][0] = hb;
  pc[0][1] = 0.0;
  pc[0][2] = 0.0;
  pc[0][3] = hb;
#pragma unroll
  for (int t = 1; t < N; ++t)
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) pc[t][mu] = s.pc[t - 1][mu];
  uint32_t leg[N];
  s.word.legs(leg);
  double a2;
  if constexpr (POL == 1) {
    double cs[N][2];
    polarisation_angles<N>(C, i, cs);
    a2 = ordered_amp2_real<N, T, true>(pc, leg, cs, tab);
  } else {
    a2 = ordered_amp2<N, T, true>(pc, leg, s.word.hel(), tab);
  }
  return finish_staged<N>(C, i, j, buf, s.word.pass(), a2, s.shat);
}

// The same from staging slot j.
template <int N, typename T = float, int POL = 0>
__device__ __forceinline__ double rec_one(const GenClass& C, int64_t i, int64_t j, const double* __restrict__ buf,
                                          RecLds<N, T>* tab) {
  Staged<N> s;
  load_staged<N>(buf, j, s);
  return rec_staged<N, T, POL>(C, i, j, buf, s, tab);
}

// The same with the event on the G lanes of a group (grouped_amp2; gdyn: the workgroup's dynamic
// LDS); with live, lane g = 0 writes the outputs and returns w, the others return 0.  slot() gives
// the event's staging slot, and is asked again after the recursion, which has no register to keep it
// in (event 0 of the launch: first); left in j.
template <int N, typename T, int G, typename F>
__device__ __forceinline__ double rec_one_g(const GenClass& C, int64_t first, const F& slot,
                                            const double* __restrict__ buf, int g, bool live, unsigned char* gdyn,
                                            int64_t& j) {
  using L = SplitLayout<N>;
  j = slot();
  const double shat = buf[L::at(j, L::kShat)];
  double pc[N][4];
  const double hb = 0.5 * (C.use_pdf ? sqrt(shat) : C.sqrt_s);
  pc[0][0] = hb;
  pc[0][1] = 0.0;
  pc[0][2] = 0.0;
  pc[0][3] = hb;
#pragma unroll
  for (int t = 1; t < N; ++t)
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) pc[t][mu] = buf[L::at(j, L::kMom + 4 * (t - 1) + mu)];
  const EventWord<N> word{(uint64_t)__double_as_longlong(buf[L::at(j, L::kMeta)])};
  uint32_t leg[N];
  word.legs(leg);
  const double a2 = grouped_amp2<N, T, G>(pc, leg, word.hel(), g, gdyn);
  if (g != 0 || !live) return 0.0;
  j = slot();
  return finish_staged<N>(C, first + j, j, buf, word.pass(), a2, shat);
}

// Launch: blockDim.x = kKinBlock, perm_lds_bytes(N, kKinBlock) bytes of dynamic LDS,
// ceil(cnt / kKinBlock) workgroups; events first .. first + cnt - 1 into slots 0 .. cnt - 1.
// Three waves per SIMD up to n = 8, two beyond (n = 12 wants 257 registers when left alone, and runs
// at one wave then: 2^20 events 204 -> 290 us).
template <int N>
__global__ __launch_bounds__(kKinBlock) __attribute__((amdgpu_waves_per_eu(N <= 8 ? 3 : 2, 8))) void k_kin(GenClass C, int64_t first, int64_t cnt, double* __restrict__ buf,
                                                   uint64_t* __restrict__ passed) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= cnt) return;
  kin_one<N>(C, first + j, j, buf, dyn_perm(), passed);
}

// Launch: blockDim.x = kLdsLanes, ceil(cnt / kLdsLanes) workgroups, first a multiple of
// kLdsLanes; workgroup b writes the partial of events first + 64 b .. (partial first / 64 + b).
// With ahead > 0 the workgroup, after issuing its own loads, pulls the staged words of tile
// blockIdx.x + ahead into the L2 cache (one 4-byte load per 128-byte line, written to a
// 256-byte LDS scrap area and never read).  Workgroups go to the XCDs in turn and one runs
// per SIMD, so with ahead a multiple of 8 and below the number resident at once, that tile
// starts on the same XCD a fraction of a workgroup's duration later and its first loads hit
// L2 instead of HBM.  Only from N = 8: the shorter workgroups of smaller N measured slower
// with it (n = 4: 0.253 against 0.238 ms per 2^22 events).
template <int N>
constexpr bool rec_prefetch() { return N >= 8; }

template <int N, typename T, int POL>
__global__ __launch_bounds__(kLdsLanes) __attribute__((amdgpu_waves_per_eu(1, rec_waves<N, T, POL>()))) void k_rec(
    GenClass C, int64_t first, int64_t cnt, const double* __restrict__ buf, double* partials, int64_t ahead,
    PassList list) {
  __shared__ RecLds<N, T> tab;
  __shared__ unsigned int scrap[rec_prefetch<N>() ? kLdsLanes : 1];
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t listed = list.count ? (int64_t)*list.count : cnt;
  if (listed < cnt) {
    if ((int64_t)blockIdx.x * blockDim.x >= listed) return;
    j = j < listed ? pass_slot<N>(buf, j) : cnt;
  }
  Staged<N> st;
  if (j < cnt) load_staged<N>(buf, j, st);
  const int64_t t = (int64_t)blockIdx.x + ahead;
  if (rec_prefetch<N>() && ahead > 0 && t * kLdsLanes < cnt) {
    // the tile's words are contiguous (SplitLayout)
    constexpr int kBytes = SplitLayout<N>::kAlways * kLdsLanes * 8;
    const char* base = reinterpret_cast<const char*>(buf + t * kLdsLanes * SplitLayout<N>::kWords);
#pragma unroll
    for (int off = 0; off < kBytes; off += kLdsLanes * 128) {
      const int o = off + (int)threadIdx.x * 128;
      if (o < kBytes)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + o),
                                         (__attribute__((address_space(3))) void*)scrap, 4, 0, 0);
    }
  }
  double w = 0.0;
  if (j < cnt) w = rec_staged<N, T, POL>(C, first + j, j, buf, st, &tab);
  if (listed < cnt) {
    if (j < cnt) list.stage[SplitLayout<N>::at(j, SplitLayout<N>::kX2)] = w;
    return;
  }
  if (partials) block_reduce_store(CSum{w, 0.0}, CSum{w * w, 0.0}, partials + 4 * (first / kLdsLanes + (int64_t)blockIdx.x));
}

// Launch: blockDim.x a multiple of 64 (at most 256), ceil(cnt G / blockDim.x) workgroups,
// grouped_lds_bytes<N, T, G>(blockDim.x) bytes of dynamic LDS, first a multiple of
// blockDim.x / G; workgroup b writes the partial of its blockDim.x / G events at
// first G / blockDim.x + b, as the one-kernel form numbers them.
template <int N, typename T, int G>
__global__ __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(group_waves<T, G>(), group_waves<T, G>()))) void k_rec_g(
    GenClass C, int64_t first, int64_t cnt, const double* __restrict__ buf, double* partials, PassList list) {
  extern __shared__ __align__(16) unsigned char gdyn[];
  int event, g;
  group_place<T, G>(event, g);
  // every lane runs the recursion (QuadSpan); those past the end repeat the last event
  const int64_t jj = (int64_t)blockIdx.x * (blockDim.x / G) + event;
  const int64_t listed = list.count ? (int64_t)*list.count : cnt;
  if ((int64_t)blockIdx.x * (blockDim.x / G) >= listed) return;
  const bool live = jj < listed;
  const auto slot = [&] {
    const double* b = buf;
    opaque(b);  // a read of its own each time
    const int64_t l = live ? jj : listed - 1;
    return listed < cnt ? pass_slot<N>(b, l) : l;
  };
  int64_t j;
  const double w = rec_one_g<N, T, G>(C, first, slot, buf, g, live, gdyn, j);
  if (listed < cnt) {
    if (g == 0 && live) list.stage[SplitLayout<N>::at(j, SplitLayout<N>::kX2)] = w;
    return;
  }
  if (partials)
    block_reduce_store(CSum{w, 0.0}, CSum{w * w, 0.0},
                       partials + 4 * (first * G / (int64_t)blockDim.x + (int64_t)blockIdx.x));
}

// The partials of k_rec (G = 1) or k_rec_g from the weights in the slots, with their launch shapes.
template <int N, typename T, int G>
__global__ __launch_bounds__(256) void k_sum_weights(int64_t first, int64_t cnt, const double* __restrict__ buf,
                                                     double* partials, const uint64_t* count) {
  if ((int64_t)*count >= cnt) return;  // every event passed: the recursion kernel wrote them
  int event = (int)threadIdx.x, g = 0;
  if constexpr (G > 1) group_place<T, G>(event, g);
  const int64_t j = (int64_t)blockIdx.x * (blockDim.x / G) + event;
  const double w = g == 0 && j < cnt ? buf[SplitLayout<N>::at(j, SplitLayout<N>::kX2)] : 0.0;
  block_reduce_store(CSum{w, 0.0}, CSum{w * w, 0.0},
                     partials + 4 * (first * G / (int64_t)blockDim.x + (int64_t)blockIdx.x));
}

// A chunk's list (after launch_pass_list); each chunk uses W.passed anew.
inline PassList pass_list(const GenWork& W) {
  return W.passed ? PassList{W.passed + W.stage_cap / 64, W.stage} : PassList{nullptr, nullptr};
}

// The kinematics kernel and the grouped recursion kernel over the class in chunks of
// W.stage_cap events (a multiple of 256); workgroups of `block` lanes.
template <int N, typename T, int G>
hipError_t launch_generate_split_g(const GenClass& C, const GenWork& W, int block, hipStream_t s) {
  if (C.count <= 0) return hipSuccess;
  if (!W.stage || W.stage_cap < 256 || W.stage_cap % 256 != 0 || block % 64 != 0 || block > 256)
    return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  for (int64_t first = 0; first < C.count && e == hipSuccess; first += W.stage_cap) {
    const int64_t cnt = std::min<int64_t>(W.stage_cap, C.count - first);
    hipLaunchKernelGGL((k_kin<N>), dim3((unsigned)((cnt + kKinBlock - 1) / kKinBlock)), dim3(kKinBlock),
                       perm_lds_bytes(N, kKinBlock), s, C, first, cnt, W.stage, W.passed);
    e = W.passed ? launch_pass_list(W, cnt, SplitLayout<N>::kX1, SplitLayout<N>::kWords, s) : hipGetLastError();
    if (e != hipSuccess) break;
    hipLaunchKernelGGL((k_rec_g<N, T, G>), dim3((unsigned)((cnt * G + block - 1) / block)), dim3(block),
                       (grouped_lds_bytes<N, T, G>(block)), s, C, first, cnt, W.stage, W.partials, pass_list(W));
    if (W.passed && W.partials)
      hipLaunchKernelGGL((k_sum_weights<N, T, G>), dim3((unsigned)((cnt * G + block - 1) / block)), dim3(block), 0, s,
                         first, cnt, W.stage, W.partials, W.passed + W.stage_cap / 64);
    e = hipGetLastError();
  }
  return e;
}

// Both kernels over the class in chunks of W.stage_cap events (a multiple of 64) through the
// caller's staging buffer; one partial per 64 events, in event order, whatever the chunking.
template <int N, typename T, int POL = 0>
hipError_t launch_generate_split(const GenClass& C, const GenWork& W, hipStream_t s) {
  if (C.count <= 0) return hipSuccess;
  if (!W.stage || W.stage_cap < kLdsLanes || W.stage_cap % kLdsLanes != 0) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  for (int64_t first = 0; first < C.count && e == hipSuccess; first += W.stage_cap) {
    const int64_t cnt = std::min<int64_t>(W.stage_cap, C.count - first);
    hipLaunchKernelGGL((k_kin<N>), dim3((unsigned)((cnt + kKinBlock - 1) / kKinBlock)), dim3(kKinBlock),
                       perm_lds_bytes(N, kKinBlock), s, C, first, cnt, W.stage, W.passed);
    e = W.passed ? launch_pass_list(W, cnt, SplitLayout<N>::kX1, SplitLayout<N>::kWords, s) : hipGetLastError();
    if (e != hipSuccess) break;
    hipLaunchKernelGGL((k_rec<N, T, POL>), dim3((unsigned)((cnt + kLdsLanes - 1) / kLdsLanes)), dim3(kLdsLanes), 0, s, C,
                       first, cnt, W.stage, W.partials, W.passed ? 0 : W.ahead, pass_list(W));
    if (W.passed && W.partials)
      hipLaunchKernelGGL((k_sum_weights<N, T, 1>), dim3((unsigned)((cnt + kLdsLanes - 1) / kLdsLanes)), dim3(kLdsLanes),
                         0, s, first, cnt, W.stage, W.partials, W.passed + W.stage_cap / 64);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace bgk
