// The fixed-order two-level reduction of per-workgroup partials (shared by every class).
#include "bg_kernels.hpp"
#include "bg_launch.hpp"

namespace bgk {

// Compensated sum of the partials [first, first + count) into (a, b) of thread 0 of the
// workgroup: lane t takes parts t, t + 256, ... in order, then a fixed butterfly and a
// fixed pass over the four waves.
__device__ __forceinline__ void group_sum(const double* __restrict__ partials, int64_t first, int64_t count, CSum& a,
                                          CSum& b) {
  a = CSum{0.0, 0.0};
  b = CSum{0.0, 0.0};
  for (int64_t p = first + threadIdx.x; p < first + count; p += blockDim.x) {
    a = cs_add(a, CSum{partials[4 * p], partials[4 * p + 1]});
    b = cs_add(b, CSum{partials[4 * p + 2], partials[4 * p + 3]});
  }
  __shared__ double red[4][4];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    CSum oa{__shfl_down(a.s, off), __shfl_down(a.c, off)};
    CSum ob{__shfl_down(b.s, off), __shfl_down(b.c, off)};
    a = cs_add(a, oa);
    b = cs_add(b, ob);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    red[wave][0] = a.s; red[wave][1] = a.c; red[wave][2] = b.s; red[wave][3] = b.c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a = CSum{red[0][0], red[0][1]};
    b = CSum{red[0][2], red[0][3]};
    for (int v = 1; v < 4; ++v) {
      a = cs_add(a, CSum{red[v][0], red[v][1]});
      b = cs_add(b, CSum{red[v][2], red[v][3]});
    }
  }
}

// Level 1: workgroup g reduces the g-th contiguous run of `per` partials.
__global__ __launch_bounds__(256) void k_finalize_runs(const double* __restrict__ partials, int64_t nparts, int64_t per,
                                                        double* level2) {
  const int64_t first = (int64_t)blockIdx.x * per;
  CSum a, b;
  group_sum(partials, first, first + per < nparts ? per : nparts - first, a, b);
  if (threadIdx.x == 0) {
    double* d = level2 + 4 * (int64_t)blockIdx.x;
    d[0] = a.s; d[1] = a.c; d[2] = b.s; d[3] = b.c;
  }
}

// Level 2 (one workgroup): the run results, in run order, are added to acc.
__global__ __launch_bounds__(256) void k_finalize(const double* __restrict__ level2, int64_t nruns, double* acc) {
  CSum a, b;
  group_sum(level2, 0, nruns, a, b);
  if (threadIdx.x == 0) {
    CSum ta{acc[0], acc[1]}, tb{acc[2], acc[3]};
    ta = cs_add(ta, a);
    tb = cs_add(tb, b);
    acc[0] = ta.s; acc[1] = ta.c; acc[2] = tb.s; acc[3] = tb.c;
  }
}

// Both levels in one workgroup of four 256-lane quarters, for at most kOneLaunchRuns runs of 256
// partials: quarter q reduces run q in the order of level 1, then the first wave takes the run
// results as level 2 does, so the sums are bitwise those of the two launches.  A launch costs 2.7 us of
// host time and leaves a gap of as much on the device; a second run for each quarter costs more
// than that (n = 4 FP32 calls with 512, 1024, 2048, 4096 partials, us: up to 16 runs in one launch
// 15.9, 16.4, 20.8, 32.1; from 5 runs in two 15.8, 16.4, 18.5, 22.9).
constexpr int kOneLaunchRuns = 4;

__global__ __launch_bounds__(1024) void k_finalize_small(const double* __restrict__ partials, int64_t nparts, double* acc) {
  __shared__ double red[16][4], run[kOneLaunchRuns][4];
  const int t = threadIdx.x & 255, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quarter = threadIdx.x >> 8;
  const int nruns = (int)((nparts + 255) / 256);
  const int64_t p = (int64_t)quarter * 256 + t;
  CSum a{0.0, 0.0}, b{0.0, 0.0};
  if (p < nparts) {
    a = cs_add(a, CSum{partials[4 * p], partials[4 * p + 1]});
    b = cs_add(b, CSum{partials[4 * p + 2], partials[4 * p + 3]});
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    a = cs_add(a, CSum{__shfl_down(a.s, off), __shfl_down(a.c, off)});
    b = cs_add(b, CSum{__shfl_down(b.s, off), __shfl_down(b.c, off)});
  }
  if (lane == 0) {
    red[wave][0] = a.s; red[wave][1] = a.c; red[wave][2] = b.s; red[wave][3] = b.c;
  }
  __syncthreads();
  if (t == 0 && quarter < nruns) {
    const int w0 = 4 * quarter;
    a = CSum{red[w0][0], red[w0][1]};
    b = CSum{red[w0][2], red[w0][3]};
    for (int v = 1; v < 4; ++v) {
      a = cs_add(a, CSum{red[w0 + v][0], red[w0 + v][1]});
      b = cs_add(b, CSum{red[w0 + v][2], red[w0 + v][3]});
    }
    double* d = run[quarter];
    d[0] = a.s; d[1] = a.c; d[2] = b.s; d[3] = b.c;
  }
  __syncthreads();
  if (wave != 0) return;
  a = b = CSum{0.0, 0.0};
  if (lane < nruns) {
    a = cs_add(a, CSum{run[lane][0], run[lane][1]});
    b = cs_add(b, CSum{run[lane][2], run[lane][3]});
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    a = cs_add(a, CSum{__shfl_down(a.s, off), __shfl_down(a.c, off)});
    b = cs_add(b, CSum{__shfl_down(b.s, off), __shfl_down(b.c, off)});
  }
  if (lane == 0) {
    const CSum ta = cs_add(CSum{acc[0], acc[1]}, a), tb = cs_add(CSum{acc[2], acc[3]}, b);
    acc[0] = ta.s; acc[1] = ta.c; acc[2] = tb.s; acc[3] = tb.c;
  }
}

hipError_t launch_finalize(const double* partials, int64_t nparts, double* level2, double* acc, hipStream_t s) {
  if (nparts <= 0) return hipSuccess;
  if (nparts <= 256 * kOneLaunchRuns) {
    hipLaunchKernelGGL(k_finalize_small, dim3(1), dim3(1024), 0, s, partials, nparts, acc);
    return hipGetLastError();
  }
  // runs of at least 256 partials, at most kFinalizeGroups runs
  int64_t per = (nparts + kFinalizeGroups - 1) / kFinalizeGroups;
  if (per < 256) per = 256;
  const int64_t nruns = (nparts + per - 1) / per;
  hipLaunchKernelGGL(k_finalize_runs, dim3((unsigned)nruns), dim3(256), 0, s, partials, nparts, per, level2);
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, level2, nruns, acc);
  return hipGetLastError();
}

// The slots of the events whose bits are set, in event order, into word `word` of the staging slots,
// and their number into *total.  A workgroup takes kListMasks masks: it adds up the masks before
// them (512 KB from L2 at most, in a chunk of 2^22 events), then each wave a share of them in turn,
// a lane per event, so that the list is written in whole lines.
constexpr int kListMasks = 256;
__global__ __launch_bounds__(1024) void k_pass_list(const uint64_t* __restrict__ masks, int64_t nmasks, double* stage,
                                                    int word, int words, uint64_t* total) {
  __shared__ int64_t before[16], own[kListMasks / 64], start[kListMasks];
  __shared__ uint64_t mask[kListMasks];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t q0 = (int64_t)blockIdx.x * kListMasks;
  int64_t sum = 0;
  for (int64_t m = tid; m < q0; m += 1024) sum += __popcll(masks[m]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) before[wave] = sum;
  const uint64_t mine = tid < kListMasks && q0 + tid < nmasks ? masks[q0 + tid] : 0;
  int64_t upto = __popcll(mine);  // inclusive over the wave's masks
  if (tid < kListMasks) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t o = __shfl_up(upto, off);
      if (lane >= off) upto += o;
    }
    start[tid] = upto - __popcll(mine);
    mask[tid] = mine;
    if (lane == 63) own[wave] = upto;
  }
  __syncthreads();
  int64_t base = 0;
#pragma unroll
  for (int v = 0; v < 16; ++v) base += before[v];
  if (blockIdx.x == gridDim.x - 1 && tid == 0) {
    uint64_t n = (uint64_t)base;
    for (int v = 0; v < kListMasks / 64; ++v) n += (uint64_t)own[v];
    *total = n;
  }
  constexpr int kShare = kListMasks / 16;
  for (int v = 0; v < wave * kShare / 64; ++v) base += own[v];
#pragma unroll 4
  for (int m = wave * kShare; m < (wave + 1) * kShare; ++m) {
    const uint64_t bits = mask[m];
    const int64_t at = base + start[m] + __popcll(bits & ((uint64_t(1) << lane) - 1));
    if ((bits >> lane) & 1)
      stage[((at >> 6) * words + word) * 64 + (at & 63)] = __longlong_as_double((q0 + m) * 64 + lane);
  }
}

hipError_t launch_pass_list(const GenWork& W, int64_t cnt, int word, int words, hipStream_t s) {
  const int64_t nmasks = (cnt + 63) / 64;
  if (nmasks <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pass_list, dim3((unsigned)((nmasks + kListMasks - 1) / kListMasks)), dim3(1024), 0, s, W.passed,
                     nmasks, W.stage, word, words, W.passed + W.stage_cap / 64);
  return hipGetLastError();
}

}  // namespace bgk
