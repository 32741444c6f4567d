// Partial records -> the solver's scalars and flags on the device: the stages
// of an iteration, run by a finalize launch (k_finalize) or, where the records
// are few, by the last workgroup of the kernel that writes them.
#pragma once

#include "wd_device.h"
#include "wd_reduce.h"

namespace wd {

__device__ __forceinline__ cx<double> cdiv(cx<double> a, cx<double> b) {
  const double d = b.re * b.re + b.im * b.im;
  return {(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}

// beta = (rho / rho_prev) (alpha / omega) of the next p-update; every finalize
// stage that changes one of its factors stores it, which keeps four FP64
// divisions out of every thread of the update.
__device__ __forceinline__ void store_beta(double* s, cx<double> rho, cx<double> rhop, cx<double> alpha,
                                           cx<double> omega) {
  const cx<double> b = cdiv(rho, rhop) * cdiv(alpha, omega);
  s[SC_BETA] = b.re;
  s[SC_BETA_IM] = b.im;
}

// Stage fa.stage of one right-hand side from its summed records v; q: its
// scalars as they were.
__device__ __forceinline__ void apply_stage(const FinArgs& fa, int rhs, const double (&v)[kWideDot], const double* q) {
  double* s = fa.sc + rhs * SC_COUNT;
  int* f = fa.fl + rhs * FL_COUNT;
  int* active = fa.active;
  int* rumask = fa.rumask;
  const int stage = fa.stage;
  const double stop = fa.tol * sqrt(q[SC_B2]);
  const cx<double> rho0 = {q[SC_RHO], q[SC_RHO + 1]}, rhop0 = {q[SC_RHOP], q[SC_RHOP + 1]};
  const cx<double> alpha0 = {q[SC_ALPHA], q[SC_ALPHA + 1]}, omega0 = {q[SC_OMEGA], q[SC_OMEGA + 1]};
  const cx<double> one = {1.0, 0.0};
  switch (stage) {
    case FIN_B2: {  // |b|; the solve then runs on b / |b| (B2 becomes 1)
      const double b2 = v[0];
      s[SC_BNORM] = sqrt(b2);
      s[SC_B2] = isfinite(b2) ? (b2 > 0.0 ? 1.0 : 0.0) : b2;
      break;
    }
    case FIN_TRUE: {  // true FP64 residual after a (re)computation of r = b - M x
      s[SC_RTRUE2] = v[0];
      s[SC_MMAX] = sqrt(v[0]);
      f[FL_CONV] = (sqrt(v[0]) <= stop) ? 1 : 0;
      if (!isfinite(v[0])) f[FL_BREAK] = stage + 1;
      // iteration resumes (an RHS that triggered the update was paused) unless done
      active[rhs] = (f[FL_CONV] || f[FL_BREAK]) ? 0 : 1;
      f[FL_RU] &= 3;  // the trigger stays as the iteration set it: the host counts the update from it
      rumask[rhs] = active[rhs];  // the residual is re-seeded only where iteration goes on
      break;
    }
    case FIN_RHO: {  // after re-encoding r: rho = <r~, r^>, |r^|^2
      s[SC_R2] = v[0];
      s[SC_RHO] = v[1];
      s[SC_RHO + 1] = v[2];
      store_beta(s, {v[1], v[2]}, rhop0, alpha0, omega0);
      break;
    }
    case FIN_TRUE_INIT:   // the same with a new shadow residual: a first iteration follows
    case FIN_TRUE_RHO: {  // both, from the residual dslash that re-encoded r itself
      s[SC_RTRUE2] = v[0];
      s[SC_MMAX] = sqrt(v[0]);
      f[FL_CONV] = (sqrt(v[0]) <= stop) ? 1 : 0;
      if (!isfinite(v[0])) f[FL_BREAK] = FIN_TRUE + 1;
      f[FL_RU] &= 3;
      active[rhs] = (f[FL_CONV] || f[FL_BREAK]) ? 0 : 1;
      rumask[rhs] = active[rhs];
      if (active[rhs]) {
        s[SC_R2] = v[1];
        s[SC_RHO] = v[2];
        s[SC_RHO + 1] = v[3];
        if (stage == FIN_TRUE_INIT) {
          s[SC_RHOP] = 1.0; s[SC_RHOP + 1] = 0.0;
          s[SC_ALPHA] = 1.0; s[SC_ALPHA + 1] = 0.0;
          s[SC_OMEGA] = 1.0; s[SC_OMEGA + 1] = 0.0;
          store_beta(s, {v[2], v[3]}, one, one, one);
        } else {
          store_beta(s, {v[2], v[3]}, rhop0, alpha0, omega0);
        }
      }
      break;
    }
    case FIN_BICG_INIT: {
      s[SC_R2] = v[0];
      s[SC_RHO] = v[1];
      s[SC_RHO + 1] = v[2];
      s[SC_RHOP] = 1.0; s[SC_RHOP + 1] = 0.0;
      s[SC_ALPHA] = 1.0; s[SC_ALPHA + 1] = 0.0;
      s[SC_OMEGA] = 1.0; s[SC_OMEGA + 1] = 0.0;
      store_beta(s, {v[1], v[2]}, one, one, one);
      break;
    }
    case FIN_BICG_ALPHA: {  // alpha = rho / <r~, v>
      ++f[FL_ITERS];
      f[FL_RU] = 0;
      const cx<double> d = {v[0], v[1]};
      if (!(d.re * d.re + d.im * d.im > 0.0) || !isfinite(d.re) || !isfinite(d.im)) {
        f[FL_BREAK] = stage + 1;
        active[rhs] = 0;
        break;
      }
      const cx<double> a = cdiv(rho0, d);
      s[SC_ALPHA] = a.re;
      s[SC_ALPHA + 1] = a.im;
      break;
    }
    case FIN_BICG_OMEGA: {  // omega = <t, s> / <t, t>
      if (v[2] == 0.0 && v[0] == 0.0 && v[1] == 0.0) {  // as in FIN_BICG_STEP
        s[SC_OMEGA] = 1.0;
        s[SC_OMEGA + 1] = 0.0;
        break;
      }
      if (!(v[2] > 0.0) || !isfinite(v[2])) {
        f[FL_BREAK] = stage + 1;
        active[rhs] = 0;
        break;
      }
      s[SC_OMEGA] = v[0] / v[2];
      s[SC_OMEGA + 1] = v[1] / v[2];
      break;
    }
    case FIN_BICG_ITER: {  // |r^|^2, <r~, r^>: beta, reliable-update trigger
      const double rn = sqrt(v[0]);
      if (!isfinite(rn) || !(omega0.re * omega0.re + omega0.im * omega0.im > 0.0)) {
        f[FL_BREAK] = stage + 1;
        active[rhs] = 0;
        break;
      }
      s[SC_RHOP] = rho0.re;
      s[SC_RHOP + 1] = rho0.im;
      s[SC_RHO] = v[1];
      s[SC_RHO + 1] = v[2];
      s[SC_R2] = v[0];
      store_beta(s, {v[1], v[2]}, rho0, alpha0, omega0);
      const double mmax = fa.restart ? q[SC_MMAX] : fmax(q[SC_MMAX], rn);
      s[SC_MMAX] = mmax;
      const int ru = rn <= stop ? 2 : (rn < fa.delta * mmax ? 1 : 0);
      f[FL_RU] = ru;
      rumask[rhs] = ru != 0;
      if (ru) active[rhs] = 0;  // paused until the host has run the update
      break;
    }
    case FIN_BICG_STEP: {
      // v = <t, s>, |t|^2, <r~, t>, <r~, s>, |s|^2 of the stored t and s:
      // omega = <t, s> / <t, t>, and for r = s - omega t at once rho = <r~, r>,
      // beta and |r|^2, so that one update can take x, r and p.  The sums are FP64
      // from the products on: against 64 bits rho, and |r|^2 down to |r| = 1e-3 |s|,
      // are closer than the FP32 sums over r that they replace.  Relative error at
      // 2,048 sites with |r| = 0.3, 0.01, 0.001 |s|, sums over r / these: |r|^2
      // 1.5e-9, 1.9e-9, 2.0e-9 / 2e-15, 1e-12, 2e-10; rho 7e-9, 3e-7, 3e-7 / 7e-16,
      // 5e-13, 7e-12 (from FP32 sums of s and t |r|^2 4e-8, 4e-5, 4e-3).
      const cx<double> ts = {v[0], v[1]}, rt = {v[3], v[4]}, rs = {v[5], v[6]};
      const double t2 = v[2], s2 = v[7];
      cx<double> om;
      if (t2 == 0.0 && ts.re == 0.0 && ts.im == 0.0) {
        // t = M_hat s = 0 means s = 0: the step already solved the system and
        // omega is arbitrary; 1 keeps the next beta finite (r becomes 0 and a
        // reliable update follows)
        om = one;
      } else if (!(t2 > 0.0) || !isfinite(t2)) {
        f[FL_BREAK] = FIN_BICG_OMEGA + 1;
        active[rhs] = 0;
        break;
      } else {
        om = {ts.re / t2, ts.im / t2};
      }
      const cx<double> oa = {(double)(float)om.re, (double)(float)om.im};  // as the update applies it
      const cx<double> rho = rs - oa * rt;
      const double r2 = s2 - 2.0 * (oa.re * ts.re + oa.im * ts.im) + (oa.re * oa.re + oa.im * oa.im) * t2;
      if (!isfinite(r2) || !isfinite(rho.re) || !isfinite(rho.im) ||
          !(om.re * om.re + om.im * om.im > 0.0)) {
        f[FL_BREAK] = FIN_BICG_ITER + 1;
        active[rhs] = 0;
        break;
      }
      s[SC_OMEGA] = om.re;
      s[SC_OMEGA + 1] = om.im;
      s[SC_RHOP] = rho0.re;
      s[SC_RHOP + 1] = rho0.im;
      s[SC_RHO] = rho.re;
      s[SC_RHO + 1] = rho.im;
      store_beta(s, rho, rho0, alpha0, om);
      const double rn = sqrt(fmax(r2, 0.0));
      s[SC_R2] = fmax(r2, 0.0);
      // reliable updates: against the largest |r^| since the last update;
      // defect correction: against the residual the inner solve started from
      const double mmax = fa.restart ? q[SC_MMAX] : fmax(q[SC_MMAX], rn);
      s[SC_MMAX] = mmax;
      // Below 2^-48 |s|^2, |r| < 6e-8 |s|, the difference and an FP32 r are rounding
      // alone: only an update can tell that from convergence
      const bool nothing_left = rn <= stop || r2 < 0x1p-48 * s2;
      const int ru = nothing_left ? 2 : (rn < fa.delta * mmax ? 1 : 0);
      f[FL_RU] = ru + 4 * (fa.step + 1);  // the update of x and r still runs (see k_bicg_xrp)
      rumask[rhs] = ru != 0;
      if (ru) active[rhs] = 0;  // paused until the host has run the update
      break;
    }
    case FIN_CG_INIT: {  // rho = |r^|^2 of the normal-equation residual; internal target
      s[SC_R2] = v[0];
      s[SC_RHO] = v[0];
      s[SC_TOLN] = fa.tol * sqrt(v[0]);
      s[SC_MMAX] = sqrt(v[0]);
      break;
    }
    case FIN_CG_ALPHA: {  // alpha = rho / |M p|^2
      ++f[FL_ITERS];
      if (!(v[0] > 0.0) || !isfinite(v[0])) {
        f[FL_BREAK] = stage + 1;
        active[rhs] = 0;
        break;
      }
      s[SC_ALPHA] = rho0.re / v[0];
      break;
    }
    case FIN_CG_ITER: {  // beta = |r_new|^2 / |r_old|^2; reliable-update trigger
      const double rn = sqrt(v[0]);
      if (!isfinite(rn)) {
        f[FL_BREAK] = stage + 1;
        active[rhs] = 0;
        break;
      }
      s[SC_RHOP] = rho0.re;
      s[SC_RHO] = v[0];
      s[SC_R2] = v[0];
      s[SC_BETA] = v[0] / rho0.re;
      const double mmax = fa.restart ? q[SC_MMAX] : fmax(q[SC_MMAX], rn);
      s[SC_MMAX] = mmax;
      const int ru = rn <= q[SC_TOLN] ? 2 : (rn < fa.delta * mmax ? 1 : 0);
      f[FL_RU] = ru;
      rumask[rhs] = ru != 0;
      if (ru) active[rhs] = 0;  // paused until the host has run the update
      break;
    }
    case FIN_CG_RHO: {  // after a reliable update: new |r^|^2, beta against the old rho
      s[SC_R2] = v[0];
      s[SC_RHO] = v[0];
      s[SC_BETA] = fa.restart ? 0.0 : v[0] / rhop0.re;  // defect correction: p = r^
      s[SC_MMAX] = sqrt(v[0]);
      break;
    }
    default: break;
  }
}

// ---- finalize inside the producing kernel -------------------------------------------
// A workgroup stores its record past its XCD's L2 (agent scope), waits for the
// store, and counts itself in; the one that completes the count reads every
// record the same way, sums them in index order and runs the stage.  No
// workgroup waits for another.  The count returns to zero for the next kernel.
// At 8^4 it saves a launch (2.7 us and the gap before it) for about 2.3 us at
// the end of the producer (x/r update 3.8 -> 5.7 us, FP64 split dslash with a
// dot 5.8 -> 8.2).  Every workgroup counts at one address, about 10 ns each: at
// 24^3x32 the x/r update's 864 took 8.7 us more against the 4.7 us saved, so
// launches of more than kFusedRecords leave the stage to k_finalize.
template <int N>
__device__ __forceinline__ bool count_record(const double (&v)[N], double* out, int rhs, int count, const FinArgs& fa) {
#pragma unroll
  for (int k = 0; k < N; ++k) __hip_atomic_store(out + k, v[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  unsigned* c = reinterpret_cast<unsigned*>(fa.sc + rhs * SC_COUNT + fa.counter);
  const unsigned before = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (before + 1 != (unsigned)count) return false;
  __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}
template <int N>
__device__ __forceinline__ void read_record(const double* rec, double (&v)[N]) {  // v += record
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] += __hip_atomic_load(rec + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int N>
__device__ __forceinline__ void wave_sum(double (&v)[N]) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] += __shfl_down(v[k], off, 64);
}

// block_sum_store of a kBlock workgroup, then the stage by the last of `count`
// workgroups of this right-hand side.  rec: the right-hand side's records.
template <int N>
__device__ __forceinline__ void block_sum_finalize(double (&d)[N], double* rec, int index, int count, int rhs,
                                                   const FinArgs& fa) {
  __shared__ double sm[kWaves][N];
  __shared__ int last;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  wave_sum<N>(d);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) sm[wid][k] = d[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    double t[N];
#pragma unroll
    for (int k = 0; k < N; ++k) t[k] = (sm[0][k] + sm[1][k]) + (sm[2][k] + sm[3][k]);
    last = count_record<N>(t, rec + index * kRecord<N>, rhs, count, fa);
  }
  __syncthreads();
  if (!last) return;
  double v[N];
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < count; i += kBlock) read_record<N>(rec + i * kRecord<N>, v);
  wave_sum<N>(v);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) sm[wid][k] = v[k];
  __syncthreads();
  if (threadIdx.x != 0) return;
  double t[kWideDot] = {};
#pragma unroll
  for (int k = 0; k < N; ++k) t[k] = (sm[0][k] + sm[1][k]) + (sm[2][k] + sm[3][k]);
  double q[SC_COUNT];
#pragma unroll
  for (int k = 0; k < SC_COUNT; ++k) q[k] = fa.sc[rhs * SC_COUNT + k];
  apply_stage(fa, rhs, t, q);
}

// The same for wave records (wave_sum_store) written by single wavefronts: a
// group of four a lane, added in the order of sum_partials, so that a split
// launch gives a solver the bits of the other shapes.
static_assert(kFusedRecords <= 4 * 64, "one group of four wave records a lane");
template <int N>
__device__ __forceinline__ void wave_sum_finalize(double (&d)[N], double* rec, int index, int count, int rhs,
                                                  const FinArgs& fa) {
  const int lane = threadIdx.x & 63;
  wave_sum<N>(d);
  int last = 0;
  if (lane == 0) last = count_record<N>(d, rec + index * kRecord<N>, rhs, count, fa);
  if (!__builtin_amdgcn_readfirstlane(last)) return;
  double q4[4][N], g[N];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int n = 0; n < N; ++n) q4[k][n] = 0.0;
    if (4 * lane < count) read_record<N>(rec + (4 * lane + k) * kRecord<N>, q4[k]);
  }
#pragma unroll
  for (int n = 0; n < N; ++n) g[n] = (q4[0][n] + q4[1][n]) + (q4[2][n] + q4[3][n]);
  wave_sum<N>(g);
  if (lane != 0) return;
  double t[kWideDot] = {};
#pragma unroll
  for (int n = 0; n < N; ++n) t[n] = g[n];
  double q[SC_COUNT];
#pragma unroll
  for (int k = 0; k < SC_COUNT; ++k) q[k] = fa.sc[rhs * SC_COUNT + k];
  apply_stage(fa, rhs, t, q);
}

}  // namespace wd
