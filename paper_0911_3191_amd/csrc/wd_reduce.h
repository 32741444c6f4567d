// Deterministic FP64 reductions: each workgroup reduces its per-site
// contributions (wavefront shuffles, then a fixed-order sum over the 4 waves
// of a 256-thread block) and writes one partial per component; a finalize
// pass sums the partials of one right-hand side in a fixed order.  No float
// atomics, so results are bitwise reproducible and do not depend on how many
// right-hand sides share a launch.
#pragma once

#include <hip/hip_runtime.h>

namespace wd {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kMaxDot = 4;  // doubles per partial record (DOT_OX below FP64: kWideDot)
constexpr int kWideDot = 8;
template <int N>
constexpr int kRecord = N > kMaxDot ? kWideDot : kMaxDot;  // record of N components

// Sum v[0..N) over the block; thread 0 writes out[0..N).  Every thread of
// the block must call it (inactive sites contribute zeros).  The LDS slots
// are shared by every call with the same N in a kernel, so the trailing
// barrier keeps a following call (the next right-hand side of a multi-RHS
// launch) from overwriting them before thread 0 has read this call's sums.
template <int N>
__device__ __forceinline__ void block_sum_store(double (&v)[N], double* out) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += __shfl_down(v[k], off, 64);
  __shared__ double sm[N][kWaves];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) sm[k][wid] = v[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = (int)blockDim.x >> 6;  // 1, 2 or 4 waves
#pragma unroll
    for (int k = 0; k < N; ++k) {
      double t = sm[k][0];
      if (nw == 2) t += sm[k][1];
      if (nw == 4) t = (sm[k][0] + sm[k][1]) + (sm[k][2] + sm[k][3]);
      out[k] = t;
    }
  }
  __syncthreads();
}

// Sum v[0..N) over one wavefront; lane 0 writes out[0..N).  The four wave
// records of 256 consecutive sites, added as (r0 + r1) + (r2 + r3), are the
// bits of block_sum_store's record of those sites.
template <int N>
__device__ __forceinline__ void wave_sum_store(double (&v)[N], double* out) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += __shfl_down(v[k], off, 64);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) out[k] = v[k];
}

// Fixed-order sum of nb partial records of N doubles (4 or 8) into res.
// Called by all kFinBlock threads of one block; the result is valid in thread
// 0.  waves: each record is four wave records (see wave_sum_store).  `before`
// runs before the barrier.
constexpr int kFinBlock = 512;
template <int N, class F>
__device__ __forceinline__ void sum_partials(const double* part, int nb, bool waves, double (&res)[N], F&& before) {
  struct Rec {
    double2 a[N / 2];
  };
  const Rec* rec = reinterpret_cast<const Rec*>(part);
  double v[N];
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = 0.0;
  if (waves) {
#pragma unroll 2
    for (int i = threadIdx.x; i < nb; i += kFinBlock) {
      const Rec r0 = rec[4 * i], r1 = rec[4 * i + 1], r2 = rec[4 * i + 2], r3 = rec[4 * i + 3];
#pragma unroll
      for (int k = 0; k < N / 2; ++k) {
        v[2 * k] += (r0.a[k].x + r1.a[k].x) + (r2.a[k].x + r3.a[k].x);
        v[2 * k + 1] += (r0.a[k].y + r1.a[k].y) + (r2.a[k].y + r3.a[k].y);
      }
    }
  } else {
#pragma unroll 4
    for (int i = threadIdx.x; i < nb; i += kFinBlock) {
      const Rec r = rec[i];
#pragma unroll
      for (int k = 0; k < N / 2; ++k) {
        v[2 * k] += r.a[k].x;
        v[2 * k + 1] += r.a[k].y;
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += __shfl_down(v[k], off, 64);
  __shared__ double sm[kFinBlock / 64][N];
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) sm[threadIdx.x >> 6][k] = v[k];
  before();
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kFinBlock / 64; ++w) t += sm[w][k];
    res[k] = t;
  }
}

}  // namespace wd
