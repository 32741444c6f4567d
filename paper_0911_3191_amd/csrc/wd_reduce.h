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
constexpr int kMaxDot = 4;  // components per partial record

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

// Fixed-order sum of nb partial records (stride kMaxDot) into res[0..4).
// Called by all kFinBlock threads of one block; the result is valid in thread
// 0.  waves: each record is four wave records (see wave_sum_store).  `before`
// runs before the barrier.
constexpr int kFinBlock = 512;
template <class F>
__device__ __forceinline__ void sum_partials(const double* part, int nb, bool waves, double (&res)[4], F&& before) {
  struct Rec {
    double2 a, b;
  };
  const Rec* rec = reinterpret_cast<const Rec*>(part);
  double2 sa = {0.0, 0.0}, sb = {0.0, 0.0};
  if (waves) {
#pragma unroll 2
    for (int i = threadIdx.x; i < nb; i += kFinBlock) {
      const Rec r0 = rec[4 * i], r1 = rec[4 * i + 1], r2 = rec[4 * i + 2], r3 = rec[4 * i + 3];
      sa.x += (r0.a.x + r1.a.x) + (r2.a.x + r3.a.x);
      sa.y += (r0.a.y + r1.a.y) + (r2.a.y + r3.a.y);
      sb.x += (r0.b.x + r1.b.x) + (r2.b.x + r3.b.x);
      sb.y += (r0.b.y + r1.b.y) + (r2.b.y + r3.b.y);
    }
  } else {
#pragma unroll 4
    for (int i = threadIdx.x; i < nb; i += kFinBlock) {
      const Rec r = rec[i];
      sa.x += r.a.x;
      sa.y += r.a.y;
      sb.x += r.b.x;
      sb.y += r.b.y;
    }
  }
  double v[4] = {sa.x, sa.y, sb.x, sb.y};
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] += __shfl_down(v[k], off, 64);
  __shared__ double sm[kFinBlock / 64][4];
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < 4; ++k) sm[threadIdx.x >> 6][k] = v[k];
  before();
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kFinBlock / 64; ++w) t += sm[w][k];
    res[k] = t;
  }
}

}  // namespace wd
