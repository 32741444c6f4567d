// Fused BLAS-1 kernels of the BiCGstab and CG iterations (Section 5.1), the
// reliable-update steps (Section 5.3, Algorithm 2) and the finalize pass
// that turns FP64 block partials into the solver's scalars on the device.
//
// Every kernel runs on a grid of (site blocks, right-hand sides); a RHS whose
// mask entry is 0 is skipped.  Per-site arithmetic is in the storage
// precision's arithmetic type (FP32 for FP32 and 16-bit fields, FP64 for
// FP64 fields); every cross-site sum is FP64 (wd_reduce.h).
#include <type_traits>

#include "wd_device.h"
#include "wd_finalize.h"

static_assert(wd::kMaxDot == wd::kMaxDotHost, "partial record size");

namespace wd {

template <typename R>
__device__ __forceinline__ cx<R> cload(const double* sc, int k) {
  return {static_cast<R>(sc[k]), static_cast<R>(sc[k + 1])};
}

// What a thread of the iteration's updates holds of a site: the whole of it,
// or (SPLIT, FP64 and FP32) three of its 16-byte chunks, the other chunks
// being other wavefronts'.  The updates are the same number by number; only
// the dot products sum in another order, which the lattice and the precision
// alone decide (blas_split), so a right-hand side's bits do not depend on its
// batch.
template <class S, bool SPLIT>
struct Part {
  using R = typename S::real;
  static constexpr int G = SPLIT ? S::NCH / 3 : 1;  // threads per site
  static constexpr int kSites = kBlock / G;         // sites per workgroup
  static constexpr int N = 12 / G;                  // complex numbers
  struct alignas(16) Chunk {
    cx<R> z[16 / sizeof(cx<R>)];
  };
  cx<R> v[N];
};
template <class S, bool SPLIT>
__device__ __forceinline__ int part_site() { return blockIdx.x * Part<S, SPLIT>::kSites + threadIdx.x % Part<S, SPLIT>::kSites; }
template <class S, bool SPLIT>
__device__ __forceinline__ void load_part(const FieldView& f, int r, int64_t i, Part<S, SPLIT>& q) {
  if constexpr (!SPLIT) {
    Spinor<typename S::real> a;
    load_spinor<S>(f, r, i, a);
#pragma unroll
    for (int n = 0; n < 12; ++n) q.v[n] = a.v[n / 3][n % 3];
  } else {
    constexpr int PER = Part<S, SPLIT>::N / 3;
    const int k0 = 3 * (threadIdx.x / Part<S, SPLIT>::kSites);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const auto c = reinterpret_cast<const typename Part<S, SPLIT>::Chunk*>(chunk_base<S>(f, r, k0 + k))[i];
#pragma unroll
      for (int j = 0; j < PER; ++j) q.v[k * PER + j] = c.z[j];
    }
  }
}
template <class S, bool SPLIT>
__device__ __forceinline__ void store_part(const FieldView& f, int r, int64_t i, const Part<S, SPLIT>& q,
                                           Part<S, SPLIT>* back = nullptr) {
  if constexpr (!SPLIT) {
    Spinor<typename S::real> a, e;
#pragma unroll
    for (int n = 0; n < 12; ++n) a.v[n / 3][n % 3] = q.v[n];
    store_spinor<S>(f, r, i, a, back ? &e : nullptr);
    if (back)
#pragma unroll
      for (int n = 0; n < 12; ++n) back->v[n] = e.v[n / 3][n % 3];
  } else {
    if (back) *back = q;
    constexpr int PER = Part<S, SPLIT>::N / 3;
    const int k0 = 3 * (threadIdx.x / Part<S, SPLIT>::kSites);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      typename Part<S, SPLIT>::Chunk c;
#pragma unroll
      for (int j = 0; j < PER; ++j) c.z[j] = q.v[k * PER + j];
      reinterpret_cast<typename Part<S, SPLIT>::Chunk*>(const_cast<char*>(chunk_base<S>(f, r, k0 + k)))[i] = c;
    }
  }
}

// ---- BiCGstab ---------------------------------------------------------------------
// p <- r + beta (p - omega v)
template <class S, bool SPLIT>
__global__ void __launch_bounds__(kBlock) k_bicg_p(int Vh, FieldView p, FieldView r, FieldView v,
                                                   const double* __restrict__ sc,
                                                   const int* __restrict__ mask) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = part_site<S, SPLIT>();
  if (i >= Vh) return;
  const double* s = sc + rhs * SC_COUNT;
  const cx<R> b = {static_cast<R>(s[SC_BETA]), static_cast<R>(s[SC_BETA_IM])};
  const cx<R> w = cload<R>(s, SC_OMEGA);
  Part<S, SPLIT> P, Rr, Vv;
  load_part<S, SPLIT>(p, rhs, i, P);
  load_part<S, SPLIT>(r, rhs, i, Rr);
  load_part<S, SPLIT>(v, rhs, i, Vv);
#pragma unroll
  for (int n = 0; n < Part<S, SPLIT>::N; ++n) P.v[n] = Rr.v[n] + b * (P.v[n] - w * Vv.v[n]);
  store_part<S, SPLIT>(p, rhs, i, P);
}

// r <- r - alpha v   (r becomes s)
template <class S, bool SPLIT>
__global__ void __launch_bounds__(kBlock) k_bicg_s(int Vh, FieldView r, FieldView v,
                                                   const double* __restrict__ sc,
                                                   const int* __restrict__ mask) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = part_site<S, SPLIT>();
  if (i >= Vh) return;
  const cx<R> al = cload<R>(sc + rhs * SC_COUNT, SC_ALPHA);
  Part<S, SPLIT> Rr, Vv;
  load_part<S, SPLIT>(r, rhs, i, Rr);
  load_part<S, SPLIT>(v, rhs, i, Vv);
#pragma unroll
  for (int n = 0; n < Part<S, SPLIT>::N; ++n) Rr.v[n] = Rr.v[n] - al * Vv.v[n];
  store_part<S, SPLIT>(r, rhs, i, Rr);
}

// x <- x + alpha p + omega s;  r <- s - omega t  (s lives in r);
// partials: |r|^2, <r~, r>
template <class S, bool SPLIT>
__global__ void __launch_bounds__(kBlock) k_bicg_xr(int Vh, FieldView x, FieldView r, FieldView p, FieldView t,
                                                    FieldView rt, const double* __restrict__ sc,
                                                    const int* __restrict__ mask, double* __restrict__ partials,
                                                    FinArgs fa) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = part_site<S, SPLIT>();
  double d[3] = {0.0, 0.0, 0.0};
  if (i < Vh) {
    const double* s = sc + rhs * SC_COUNT;
    const cx<R> al = cload<R>(s, SC_ALPHA), om = cload<R>(s, SC_OMEGA);
    Part<S, SPLIT> X, Ss, P, T, Rt;
    load_part<S, SPLIT>(x, rhs, i, X);
    load_part<S, SPLIT>(r, rhs, i, Ss);
    load_part<S, SPLIT>(p, rhs, i, P);
    load_part<S, SPLIT>(t, rhs, i, T);
    load_part<S, SPLIT>(rt, rhs, i, Rt);
    R nn = 0, re = 0, im = 0;
#pragma unroll
    for (int n = 0; n < Part<S, SPLIT>::N; ++n) {
      X.v[n] = X.v[n] + al * P.v[n] + om * Ss.v[n];
      const cx<R> rn = Ss.v[n] - om * T.v[n];
      Ss.v[n] = rn;
      nn += rn.re * rn.re + rn.im * rn.im;
      const cx<R> q = cmulc(Rt.v[n], rn);
      re += q.re;
      im += q.im;
    }
    store_part<S, SPLIT>(x, rhs, i, X);
    store_part<S, SPLIT>(r, rhs, i, Ss);
    d[0] = nn;
    d[1] = re;
    d[2] = im;
  }
  double* rec = partials + (int64_t)rhs * gridDim.x * kMaxDot;
  if (fa.stage < 0) block_sum_store<3>(d, rec + blockIdx.x * kMaxDot);
  else block_sum_finalize<3>(d, rec, blockIdx.x, gridDim.x, rhs, fa);
}

// x <- x + alpha p + omega s;  r <- s - omega t  (s lives in r);
// p <- r + beta (p - omega v), unless the right-hand side pauses for a
// reliable update, which re-seeds r first.  Eight fields moved; as an x/r update
// with <r~, r> and |r|^2 and a p update it was eleven (and two launches more),
// see FIN_BICG_STEP.  32^3x64, binary16, 12 RHS: 956 us (5.6 TB/s) instead of
// 888 + 488; the launch that now also reads r~ and sums in FP64 takes 806
// instead of 604.  FP64 fields keep the two updates (k_bicg_xr, k_bicg_p).
template <class S, bool SPLIT>
__global__ void __launch_bounds__(kBlock) k_bicg_xrp(int Vh, FieldView x, FieldView r, FieldView p, FieldView t,
                                                     FieldView v, const double* __restrict__ sc,
                                                     const int* __restrict__ fl, int step) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  const int ru = fl[rhs * FL_COUNT + FL_RU];
  if (ru >> 2 != step + 1) return;
  const bool go_on = (ru & 3) == 0;
  const int i = part_site<S, SPLIT>();
  if (i >= Vh) return;
  const double* s = sc + rhs * SC_COUNT;
  const cx<R> al = cload<R>(s, SC_ALPHA), om = cload<R>(s, SC_OMEGA);
  const cx<R> b = {static_cast<R>(s[SC_BETA]), static_cast<R>(s[SC_BETA_IM])};
  Part<S, SPLIT> X, Ss, P, T, Vv;
  load_part<S, SPLIT>(x, rhs, i, X);
  load_part<S, SPLIT>(r, rhs, i, Ss);
  load_part<S, SPLIT>(p, rhs, i, P);
  load_part<S, SPLIT>(t, rhs, i, T);
  if (go_on) load_part<S, SPLIT>(v, rhs, i, Vv);
#pragma unroll
  for (int n = 0; n < Part<S, SPLIT>::N; ++n) {
    X.v[n] = X.v[n] + al * P.v[n] + om * Ss.v[n];
    Ss.v[n] = Ss.v[n] - om * T.v[n];
  }
  store_part<S, SPLIT>(x, rhs, i, X);
  Part<S, SPLIT> Rr;  // p follows the stored r
  store_part<S, SPLIT>(r, rhs, i, Ss, &Rr);
  if (!go_on) return;
#pragma unroll
  for (int n = 0; n < Part<S, SPLIT>::N; ++n) P.v[n] = Rr.v[n] + b * (P.v[n] - om * Vv.v[n]);
  store_part<S, SPLIT>(p, rhs, i, P);
}

// ---- CG on the normal equations ---------------------------------------------------
// x <- x + alpha p;  r <- r - alpha q;  partials: |r|^2
template <class S, bool SPLIT>
__global__ void __launch_bounds__(kBlock) k_cg_xr(int Vh, FieldView x, FieldView r, FieldView p,
                                                  FieldView q, const double* __restrict__ sc,
                                                  const int* __restrict__ mask,
                                                  double* __restrict__ partials, FinArgs fa) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = part_site<S, SPLIT>();
  double d[1] = {0.0};
  if (i < Vh) {
    const R al = static_cast<R>(sc[rhs * SC_COUNT + SC_ALPHA]);
    Part<S, SPLIT> X, Rr, P, Q;
    load_part<S, SPLIT>(x, rhs, i, X);
    load_part<S, SPLIT>(r, rhs, i, Rr);
    load_part<S, SPLIT>(p, rhs, i, P);
    load_part<S, SPLIT>(q, rhs, i, Q);
    R nn = 0;
#pragma unroll
    for (int n = 0; n < Part<S, SPLIT>::N; ++n) {
      X.v[n] = X.v[n] + al * P.v[n];
      Rr.v[n] = Rr.v[n] - al * Q.v[n];
      nn += Rr.v[n].re * Rr.v[n].re + Rr.v[n].im * Rr.v[n].im;
    }
    store_part<S, SPLIT>(x, rhs, i, X);
    store_part<S, SPLIT>(r, rhs, i, Rr);
    d[0] = nn;
  }
  double* rec = partials + (int64_t)rhs * gridDim.x * kMaxDot;
  if (fa.stage < 0) block_sum_store<1>(d, rec + blockIdx.x * kMaxDot);
  else block_sum_finalize<1>(d, rec, blockIdx.x, gridDim.x, rhs, fa);
}

// p <- r + beta p
template <class S, bool SPLIT>
__global__ void __launch_bounds__(kBlock) k_cg_p(int Vh, FieldView p, FieldView r,
                                                 const double* __restrict__ sc,
                                                 const int* __restrict__ mask) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = part_site<S, SPLIT>();
  if (i >= Vh) return;
  const R be = static_cast<R>(sc[rhs * SC_COUNT + SC_BETA]);
  Part<S, SPLIT> P, Rr;
  load_part<S, SPLIT>(p, rhs, i, P);
  load_part<S, SPLIT>(r, rhs, i, Rr);
#pragma unroll
  for (int n = 0; n < Part<S, SPLIT>::N; ++n) P.v[n] = Rr.v[n] + be * P.v[n];
  store_part<S, SPLIT>(p, rhs, i, P);
}

// ---- generic field operations -----------------------------------------------------
// dst (precision D) <- src (precision S), re-encoding per site.
template <class D, class S>
__global__ void __launch_bounds__(kBlock) k_convert(int Vh, FieldView dst, FieldView src,
                                                    const int* __restrict__ mask) {
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Vh) return;
  Spinor<typename S::real> a;
  load_spinor<S>(src, rhs, i, a);
  Spinor<typename D::real> b;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      b.v[s][c] = {static_cast<typename D::real>(a.v[s][c].re), static_cast<typename D::real>(a.v[s][c].im)};
  store_spinor<D>(dst, rhs, i, b);
}

template <class S>
__global__ void __launch_bounds__(kBlock) k_zero(int Vh, FieldView f, const int* __restrict__ mask) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Vh) return;
  Spinor<R> z;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) z.v[s][c] = {R(0), R(0)};
  store_spinor<S>(f, rhs, i, z);
}

// partials: |f|^2
template <class S>
__global__ void __launch_bounds__(kBlock) k_norm2(int Vh, FieldView f, const int* __restrict__ mask,
                                                  double* __restrict__ partials) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  double d[1] = {0.0};
  if (i < Vh) {
    Spinor<R> a;
    load_spinor<S>(f, rhs, i, a);
    R nn = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) nn += a.v[s][c].re * a.v[s][c].re + a.v[s][c].im * a.v[s][c].im;
    d[0] = nn;
  }
  block_sum_store<1>(d, partials + ((int64_t)rhs * gridDim.x + blockIdx.x) * kMaxDot);
}

// ---- reliable update ----------------------------------------------------------------
// x (FP64) <- x + xh (low precision, decoded): the groupwise solution update.
template <class S>
__global__ void __launch_bounds__(kBlock) k_accum(int Vh, FieldView x, FieldView xh,
                                                  const int* __restrict__ mask) {
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Vh) return;
  Spinor<double> X;
  Spinor<typename S::real> H;
  load_spinor<SF64>(x, rhs, i, X);
  load_spinor<S>(xh, rhs, i, H);
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      X.v[s][c] = X.v[s][c] + cx<double>{static_cast<double>(H.v[s][c].re), static_cast<double>(H.v[s][c].im)};
  store_spinor<SF64>(x, rhs, i, X);
}

// partials: |b|^2 of a canonical full-lattice FP64 array [nrhs][2 Vh][24] read
// as 16-byte pairs in address order: block k sums pairs [24 kBlock k,
// 24 kBlock (k + 1)) of its RHS (the reals of 2 kBlock sites), so a RHS has as
// many records as the other BLAS-1 kernels.
__global__ void __launch_bounds__(kBlock) k_canon_norm2(int Vh, const double* __restrict__ canon,
                                                        double* __restrict__ partials) {
  const int rhs = blockIdx.y;
  const int64_t npair = 24 * (int64_t)Vh;  // 16-byte pairs per RHS
  const double2* src = reinterpret_cast<const double2*>(canon) + (int64_t)rhs * npair;
  const int64_t j0 = (int64_t)blockIdx.x * 24 * kBlock + threadIdx.x;
  double nn = 0.0;
#pragma unroll 4
  for (int k = 0; k < 24; ++k) {
    const int64_t j = j0 + (int64_t)k * kBlock;
    if (j < npair) {
      const double2 v = src[j];
      nn += v.x * v.x + v.y * v.y;
    }
  }
  double d[1] = {nn};
  block_sum_store<1>(d, partials + ((int64_t)rhs * gridDim.x + blockIdx.x) * kMaxDot);
}

// rh <- enc(r64); xh <- 0; partials: |rh|^2, <rt, rh> (has_rt = 0: no rt;
// 1: rt read; 2: rt <- enc(r64) too, the shadow residual of a fresh start).
template <class S>
__global__ void __launch_bounds__(kBlock) k_reencode(int Vh, FieldView rh, FieldView xh, FieldView r64,
                                                     FieldView rt, int has_rt,
                                                     const int* __restrict__ mask,
                                                     double* __restrict__ partials) {
  using R = typename S::real;
  const int rhs = blockIdx.y;
  if (mask && !mask[rhs]) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  double d[3] = {0.0, 0.0, 0.0};
  if (i < Vh) {
    Spinor<double> a;
    load_spinor<SF64>(r64, rhs, i, a);
    Spinor<R> b, z;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        b.v[s][c] = {static_cast<R>(a.v[s][c].re), static_cast<R>(a.v[s][c].im)};
        z.v[s][c] = {R(0), R(0)};
      }
    R nn = 0, re = 0, im = 0;
    Spinor<R> t, e = b;
    if (has_rt == 1) load_spinor<S>(rt, rhs, i, t);
    store_spinor<S>(rh, rhs, i, e, &b);  // the dots see the stored (re-encoded) residual
    if (has_rt == 2) {
      store_spinor<S>(rt, rhs, i, e);
      t = b;
    }
    store_spinor<S>(xh, rhs, i, z);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        nn += b.v[s][c].re * b.v[s][c].re + b.v[s][c].im * b.v[s][c].im;
        if (has_rt) {
          const cx<R> q = cmulc(t.v[s][c], b.v[s][c]);
          re += q.re;
          im += q.im;
        }
      }
    d[0] = nn;
    d[1] = re;
    d[2] = im;
  }
  block_sum_store<3>(d, partials + ((int64_t)rhs * gridDim.x + blockIdx.x) * kMaxDot);
}

// ---- finalize: partials -> scalars ---------------------------------------------------
// What bounds it is latency: the records come from other XCDs, and one CU has
// only so many misses in flight.  The records of a right-hand side are summed
// by gridDim.x workgroups, each a range of `chunk`; the last of them adds the
// sums in order (see count_record) and runs the stage.  24^3x32, 864 records of
// four wave records: 11.0 us with one workgroup for records of 8 doubles and 6.0
// of 4, with seven 7.6 and 5.4.  8^4 (one workgroup) 2.7 us.
template <int N>
__global__ void __launch_bounds__(kFinBlock) k_finalize(int nb, int chunk, int waves,
                                                        const double* __restrict__ partials, double* sums,
                                                        const int* __restrict__ mask, FinArgs fa) {
  const int rhs = blockIdx.y, count = gridDim.x;
  if (mask && !mask[rhs]) return;
  const double* s = fa.sc + rhs * SC_COUNT;
  __shared__ double q[SC_COUNT];  // the scalars as they were
  const double own = threadIdx.x < SC_COUNT ? s[threadIdx.x] : 0.0;
  double r[N], v[kWideDot] = {};  // a stage reads the components that its records have
  const int first = blockIdx.x * chunk;
  sum_partials<N>(partials + ((int64_t)rhs * nb + first) * (waves ? 4 : 1) * N, min(chunk, nb - first), waves != 0, r,
                  [&] { if (threadIdx.x < SC_COUNT) q[threadIdx.x] = own; });
  if (threadIdx.x >= 64) return;
  if (count > 1) {
    sums += (int64_t)rhs * count * N;
    int last = 0;
    if (threadIdx.x == 0) last = count_record<N>(r, sums + blockIdx.x * N, rhs, count, fa);
    if (!__builtin_amdgcn_readfirstlane(last)) return;
#pragma unroll
    for (int k = 0; k < N; ++k) r[k] = 0.0;
    if ((int)threadIdx.x < count) read_record<N>(sums + threadIdx.x * N, r);
    wave_sum<N>(r);
  }
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = r[k];
  apply_stage(fa, rhs, v, q);
}

// CG stopping: at a reliable update the true residual |r| of M_hat x = b_hat is
// known; if it misses tol |b| the internal target on the normal-equation
// residual is tightened by the ratio.  Runs after FIN_TRUE.
__global__ void k_cg_tighten(int nrhs, double* sc, const int* fl, const int* mask, double tol) {
  const int rhs = blockIdx.x * blockDim.x + threadIdx.x;
  if (rhs >= nrhs || (mask && !mask[rhs])) return;
  double* s = sc + rhs * SC_COUNT;
  if (fl[rhs * FL_COUNT + FL_CONV]) return;
  const double stop = tol * sqrt(s[SC_B2]);
  const double rt = sqrt(s[SC_RTRUE2]);
  if (rt > stop) s[SC_TOLN] = fmin(s[SC_TOLN], s[SC_TOLN] * stop / rt);
}

__global__ void k_init_flags(int nrhs, int* fl, int* active, int* rumask, double* sc, int counter) {
  const int rhs = blockIdx.x * blockDim.x + threadIdx.x;
  if (rhs >= nrhs) return;
  sc[rhs * SC_COUNT + counter] = 0.0;  // FinArgs::counter: zero bits
  for (int k = 0; k < FL_COUNT; ++k) fl[rhs * FL_COUNT + k] = 0;
  active[rhs] = 1;
  rumask[rhs] = 1;
}

// ---- launchers ----------------------------------------------------------------------------
template <class Fn>
static hipError_t by_prec(wd_prec p, Fn&& fn) {
  switch (p) {
    case WD_FP64: fn(SF64{}); break;
    case WD_FP32: fn(SF32{}); break;
    case WD_HALF_I16: fn(SI16{}); break;
    case WD_HALF_F16: fn(SF16{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

static FieldView fv(const Field& f) { return FieldView{f.ptr, f.stride, f.nrhs}; }
static dim3 grid_of(const Geom& g, int nrhs) { return dim3((g.Vh + kBlock - 1) / kBlock, nrhs); }

// Where the updates of an iteration split a site over threads: FP64 and FP32
// lattices whose whole-site launch leaves most of the chip idle, each thread
// of it with up to 60 loads of its own.  8^4 FP64, microseconds: p 4.0 -> 2.9, s 4.1 -> 2.4,
// x/r 6.3 -> 3.8.
static bool blas_split(const Geom& g, wd_prec p) { return !is_half(p) && g.Vh <= 65536; }
int blas_dot_records(const Geom& g, wd_prec p) {
  const int sites = blas_split(g, p) ? kBlock * 3 / spinor_chunks(p) : kBlock;
  return (g.Vh + sites - 1) / sites;
}
template <class S, class Fn>
static void by_split(const Geom& g, int nrhs, Fn&& fn) {
  const dim3 grid(blas_dot_records(g, S::prec), nrhs);
  if constexpr (!kHalf<S>) {
    if (blas_split(g, S::prec)) return fn(grid, std::true_type{});
  }
  fn(grid, std::false_type{});
}

hipError_t blas_bicg_p(const Geom& g, wd_prec pr, Field p, Field r, Field v, const double* sc,
                       const int* mask, hipStream_t s) {
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    by_split<S>(g, p.nrhs, [&](dim3 grid, auto split) {
      k_bicg_p<S, decltype(split)::value><<<grid, kBlock, 0, s>>>(g.Vh, fv(p), fv(r), fv(v), sc, mask);
    });
  });
}

hipError_t blas_bicg_s(const Geom& g, wd_prec pr, Field r, Field v, const double* sc,
                       const int* mask, hipStream_t s) {
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    by_split<S>(g, r.nrhs, [&](dim3 grid, auto split) {
      k_bicg_s<S, decltype(split)::value><<<grid, kBlock, 0, s>>>(g.Vh, fv(r), fv(v), sc, mask);
    });
  });
}

hipError_t blas_bicg_xrp(const Geom& g, wd_prec pr, Field x, Field r, Field p, Field t, Field v, const double* sc,
                         const int* fl, int step, hipStream_t s) {
  if (pr == WD_FP64) return hipErrorInvalidValue;  // blas_bicg_xr
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    if constexpr (S::prec != WD_FP64)
      by_split<S>(g, x.nrhs, [&](dim3 grid, auto split) {
        k_bicg_xrp<S, decltype(split)::value><<<grid, kBlock, 0, s>>>(g.Vh, fv(x), fv(r), fv(p), fv(t), fv(v), sc, fl,
                                                                      step);
      });
  });
}

hipError_t blas_bicg_xr(const Geom& g, Field x, Field r, Field p, Field t, Field rt, const double* sc,
                        const int* mask, double* partials, const FinArgs& fa, hipStream_t s) {
  by_split<SF64>(g, x.nrhs, [&](dim3 grid, auto split) {
    k_bicg_xr<SF64, decltype(split)::value><<<grid, kBlock, 0, s>>>(g.Vh, fv(x), fv(r), fv(p), fv(t), fv(rt), sc,
                                                                   mask, partials, fa);
  });
  return hipGetLastError();
}

hipError_t blas_cg_xr(const Geom& g, wd_prec pr, Field x, Field r, Field p, Field q,
                      const double* sc, const int* mask, double* partials, const FinArgs& fa, hipStream_t s) {
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    by_split<S>(g, x.nrhs, [&](dim3 grid, auto split) {
      k_cg_xr<S, decltype(split)::value><<<grid, kBlock, 0, s>>>(g.Vh, fv(x), fv(r), fv(p), fv(q), sc, mask,
                                                                 partials, fa);
    });
  });
}

hipError_t blas_cg_p(const Geom& g, wd_prec pr, Field p, Field r, const double* sc,
                     const int* mask, hipStream_t s) {
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    by_split<S>(g, p.nrhs, [&](dim3 grid, auto split) {
      k_cg_p<S, decltype(split)::value><<<grid, kBlock, 0, s>>>(g.Vh, fv(p), fv(r), sc, mask);
    });
  });
}

hipError_t blas_convert(const Geom& g, wd_prec dst_prec, Field dst, wd_prec src_prec, Field src,
                        const int* mask, hipStream_t s) {
  return by_prec(dst_prec, [&](auto dtag) {
    using D = decltype(dtag);
    (void)by_prec(src_prec, [&](auto stag) {
      using S = decltype(stag);
      k_convert<D, S><<<grid_of(g, dst.nrhs), kBlock, 0, s>>>(g.Vh, fv(dst), fv(src), mask);
    });
  });
}

hipError_t blas_zero(const Geom& g, wd_prec pr, Field f, const int* mask, hipStream_t s) {
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    k_zero<S><<<grid_of(g, f.nrhs), kBlock, 0, s>>>(g.Vh, fv(f), mask);
  });
}

hipError_t blas_norm2(const Geom& g, wd_prec pr, Field f, const int* mask, double* partials,
                      hipStream_t s) {
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    k_norm2<S><<<grid_of(g, f.nrhs), kBlock, 0, s>>>(g.Vh, fv(f), mask, partials);
  });
}

hipError_t blas_accum(const Geom& g, wd_prec pr, Field x64, Field xh, const int* mask, hipStream_t s) {
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    k_accum<S><<<grid_of(g, x64.nrhs), kBlock, 0, s>>>(g.Vh, fv(x64), fv(xh), mask);
  });
}

hipError_t blas_canon_norm2(const Geom& g, const double* canon, int nrhs, double* partials, hipStream_t s) {
  k_canon_norm2<<<grid_of(g, nrhs), kBlock, 0, s>>>(g.Vh, canon, partials);
  return hipGetLastError();
}

hipError_t blas_reencode(const Geom& g, wd_prec pr, Field rh, Field xh, Field r64, const Field* rt,
                         const int* mask, double* partials, hipStream_t s, bool set_rt) {
  if (set_rt && !rt) return hipErrorInvalidValue;
  return by_prec(pr, [&](auto tag) {
    using S = decltype(tag);
    k_reencode<S><<<grid_of(g, rh.nrhs), kBlock, 0, s>>>(g.Vh, fv(rh), fv(xh), fv(r64),
                                                         rt ? fv(*rt) : FieldView{nullptr, 0, 0},
                                                         rt ? (set_rt ? 2 : 1) : 0, mask, partials);
  });
}

// Workgroups of k_finalize: by the records alone, so that every launch shape of
// the kernel before it gives the same sums.  128 records to a workgroup and 64
// take the same time (24^3x32: 7.6 and 5.4 us both).
constexpr int kFinChunk = 128, kFinGroups = 32;
static_assert(kFinGroups <= 64, "one sum a lane");

hipError_t solver_finalize(const FinArgs& fa, int nrhs, int nb, int waves, const double* partials, double* sums,
                           const int* mask, hipStream_t s) {
  int groups = !sums || nb <= kFusedRecords ? 1 : (nb + kFinChunk - 1) / kFinChunk;
  if (groups > kFinGroups) groups = kFinGroups;
  const int chunk = (nb + groups - 1) / groups;
  const dim3 grid((nb + chunk - 1) / chunk, nrhs);
  if (fa.stage == FIN_BICG_STEP) k_finalize<kWideDot><<<grid, kFinBlock, 0, s>>>(nb, chunk, waves, partials, sums, mask, fa);
  else k_finalize<kMaxDot><<<grid, kFinBlock, 0, s>>>(nb, chunk, waves, partials, sums, mask, fa);
  return hipGetLastError();
}

hipError_t solver_cg_tighten(int nrhs, double* sc, const int* fl, const int* mask, double tol,
                             hipStream_t s) {
  k_cg_tighten<<<(nrhs + 63) / 64, 64, 0, s>>>(nrhs, sc, fl, mask, tol);
  return hipGetLastError();
}

hipError_t solver_init_flags(int nrhs, int* fl, int* active, int* rumask, double* sc, int counter, hipStream_t s) {
  k_init_flags<<<(nrhs + 63) / 64, 64, 0, s>>>(nrhs, fl, active, rumask, sc, counter);
  return hipGetLastError();
}

}  // namespace wd
