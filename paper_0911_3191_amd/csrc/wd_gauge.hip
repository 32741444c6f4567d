// Gauge-field preprocessing on the device, all in FP64:
//  - the 8-real link format (Appendix A.2): a2, a3, b1 and the phases of a1
//    and c1, written in every storage precision of the handle;
//  - the temporal gauge of Section 4.3: g(x,0) = 1, g(x,t+1) = g(x,t) U_t(x,t)
//    along each time line, U'_mu(x) = g(x) U_mu(x) g(x+mu)^dagger, so that
//    every temporal link but those of the last time slice is the unit
//    matrix; spinors rotate as psi'(x) = g(x) psi(x);
//  - the check that a field handed in as temporal-gauge really is one.
#include "wd_device.h"

namespace wd {

namespace {

struct Lat {
  int L[4];
  int Lxh, Vh;
  int64_t V;
};

Lat lat_of(const Geom& g) {
  Lat l;
  for (int k = 0; k < 4; ++k) l.L[k] = g.L[k];
  l.Lxh = g.Lxh;
  l.Vh = g.Vh;
  l.V = 2 * (int64_t)g.Vh;
  return l;
}

// Parity of lexicographic site L; its checkerboard index is L / 2 (Lx is even).
__device__ __forceinline__ int parity_of(const Lat& m, int L) {
  const int row = L / m.L[0];
  const int x = L - row * m.L[0];
  const int y = row % m.L[1];
  const int zt = row / m.L[1];
  return (x + y + zt % m.L[2] + zt / m.L[2]) & 1;
}

// 3x3 complex products on [3][3][re,im] arrays in registers.
__device__ __forceinline__ void mm(const double (&A)[18], const double (&B)[18], double (&C)[18]) {  // C = A B
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double re = 0.0, im = 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double ar = A[6 * i + 2 * k], ai = A[6 * i + 2 * k + 1];
        const double br = B[6 * k + 2 * j], bi = B[6 * k + 2 * j + 1];
        re += ar * br - ai * bi;
        im += ar * bi + ai * br;
      }
      C[6 * i + 2 * j] = re;
      C[6 * i + 2 * j + 1] = im;
    }
}
__device__ __forceinline__ void mmd(const double (&A)[18], const double (&B)[18], double (&C)[18]) {  // C = A B^dagger
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double re = 0.0, im = 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double ar = A[6 * i + 2 * k], ai = A[6 * i + 2 * k + 1];
        const double br = B[6 * j + 2 * k], bi = -B[6 * j + 2 * k + 1];
        re += ar * br - ai * bi;
        im += ar * bi + ai * br;
      }
      C[6 * i + 2 * j] = re;
      C[6 * i + 2 * j + 1] = im;
    }
}
__device__ __forceinline__ void load9(const double2* p, double (&A)[18]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 v = p[k];
    A[2 * k] = v.x;
    A[2 * k + 1] = v.y;
  }
}

// One thread per (site, mu): the 8 reals of U[lex][mu] in every precision of
// the handle.  16-bit: the phases are stored divided by pi, so all 8 values
// lie in [-1, 1] and use the link encoding of the 12-real format.
__global__ void __launch_bounds__(kLinkThreads) gauge_encode8_kernel(Lat m, const double* __restrict__ U,
                                                                     int64_t stride, char* f64, char* f32, char* i16,
                                                                     char* h16) {
  __shared__ LinkTile tile;
  const int L0 = blockIdx.x * kLinkSites;
  const int n = min(kLinkSites, 2 * m.Vh - L0);
  load_links(U, L0, n, tile);
  __syncthreads();
  const int site = threadIdx.x & 63, mu = threadIdx.x >> 6;
  if (site >= n) return;
  const int par = parity_of(m, L0 + site), cb = (L0 + site) >> 1;
  const double* u = reinterpret_cast<const double*>(link_record(tile, mu, site));
  double v[8] = {u[2], u[3], u[4], u[5], u[6], u[7], atan2(u[1], u[0]), atan2(u[13], u[12])};
  const int64_t chunk = (int64_t)(par * 4 + mu);
  if (f64) {
    for (int k = 0; k < 4; ++k)
      reinterpret_cast<double2*>(f64 + ((chunk * 4 + k) * stride) * 16)[cb] = make_double2(v[2 * k], v[2 * k + 1]);
  }
  if (f32) {
    for (int k = 0; k < 2; ++k)
      reinterpret_cast<float4*>(f32 + ((chunk * 2 + k) * stride) * 16)[cb] =
          make_float4((float)v[4 * k], (float)v[4 * k + 1], (float)v[4 * k + 2], (float)v[4 * k + 3]);
  }
  double w[8];
  for (int k = 0; k < 8; ++k) w[k] = (k < 6) ? v[k] : v[k] * (1.0 / M_PI);
  if (i16) {
    uint32_t q[4];
    for (int j = 0; j < 4; ++j) {
      const float a = fminf(fmaxf(rintf((float)w[2 * j] * 32767.0f), -32767.0f), 32767.0f);
      const float b = fminf(fmaxf(rintf((float)w[2 * j + 1] * 32767.0f), -32767.0f), 32767.0f);
      q[j] = (uint32_t)(uint16_t)(int16_t)a | ((uint32_t)(uint16_t)(int16_t)b << 16);
    }
    reinterpret_cast<uint4*>(i16 + (chunk * stride) * 16)[cb] = make_uint4(q[0], q[1], q[2], q[3]);
  }
  if (h16) {
    uint32_t q[4];
    for (int j = 0; j < 4; ++j)
      q[j] = (uint32_t)f_to_h16(pin_f32((float)w[2 * j])) | ((uint32_t)f_to_h16(pin_f32((float)w[2 * j + 1])) << 16);
    reinterpret_cast<uint4*>(h16 + (chunk * stride) * 16)[cb] = make_uint4(q[0], q[1], q[2], q[3]);
  }
}

// Largest |U_t(x) - 1| (max norm) over the temporal links of t < Lt - 1, as the
// bits of a non-negative double (their order is that of the values).  Nine
// lanes share a link, 16 bytes each; one atomic per workgroup (24^3x32: 88 ->
// 35 us).
constexpr int kCheckIters = 8;
__global__ void __launch_bounds__(256) temporal_check_kernel(Lat m, const double* __restrict__ U,
                                                             unsigned long long* dev) {
  const int64_t pieces = (m.V - (int64_t)m.L[0] * m.L[1] * m.L[2]) * 9;  // sites of t < Lt - 1
  const double2* src = reinterpret_cast<const double2*>(U);
  double d = 0.0;
#pragma unroll
  for (int k = 0; k < kCheckIters; ++k) {
    const int64_t j = ((int64_t)blockIdx.x * kCheckIters + k) * 256 + threadIdx.x;
    const int64_t i = min(j, pieces - 1);
    const int64_t site = i / 9;
    const int part = (int)(i - site * 9);
    const double2 v = src[site * 36 + 27 + part];
    const double one = (part == 0 || part == 4 || part == 8) ? 1.0 : 0.0;  // the diagonal's real parts
    const double a = fabs(v.x - one), b = fabs(v.y);
    d = fmax(d, !(a <= 1e300) || !(b <= 1e300) ? 1e300 : fmax(a, b));  // NaN or Inf counts as far from 1
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) d = fmax(d, __shfl_down(d, off, 64));
  __shared__ double sm[4];
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = d;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(dev, (unsigned long long)__double_as_longlong(fmax(fmax(sm[0], sm[1]), fmax(sm[2], sm[3]))));
}

// g along each time line.  The rows of g(t + 1) = g(t) U_t(t) are independent:
// one thread per (spatial site, row), which shares its link with two
// neighbouring lanes and has the links of the next two time slices in flight
// (the chain of Lt products is otherwise a chain of memory latencies:
// 24^3x32 95 -> 53 us).
__global__ void __launch_bounds__(128) temporal_g_kernel(Lat m, const double* __restrict__ U,
                                                         double* __restrict__ g) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t V3 = (int64_t)m.L[0] * m.L[1] * m.L[2];
  if (i >= V3 * 3) return;
  const int64_t s = i / 3;
  const int row = (int)(i - 3 * s);
  const double2* src = reinterpret_cast<const double2*>(U) + s * 36 + 27;
  const int64_t slice = V3 * 36;
  const int last = m.L[3] - 2;  // the last link that a later site needs
  double cur[6], b0[18], b1[18];
#pragma unroll
  for (int k = 0; k < 6; ++k) cur[k] = (k == 2 * row) ? 1.0 : 0.0;
  load9(src, b0);
  load9(src + slice * min(1, last), b1);
  for (int t = 0; t < m.L[3]; ++t) {
    double2* dst = reinterpret_cast<double2*>(g) + (s + V3 * t) * 9 + 3 * row;
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[k] = make_double2(cur[2 * k], cur[2 * k + 1]);
    if (t > last) break;
    double nxt[6];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double re = 0.0, im = 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double ar = cur[2 * k], ai = cur[2 * k + 1];
        const double br = b0[6 * k + 2 * j], bi = b0[6 * k + 2 * j + 1];
        re += ar * br - ai * bi;
        im += ar * bi + ai * br;
      }
      nxt[2 * j] = re;
      nxt[2 * j + 1] = im;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) cur[k] = nxt[k];
#pragma unroll
    for (int k = 0; k < 18; ++k) b0[k] = b1[k];
    load9(src + slice * min(t + 2, last), b1);
  }
}

// U'_mu(x) = g(x) U_mu(x) g(x + mu)^dagger: one thread per (site, mu), links
// and g(x) through LDS.  Uo may alias U (a workgroup has read its links
// before it writes them).  24^3x32: 213 -> 106 us.
__global__ void __launch_bounds__(kLinkThreads) temporal_links_kernel(Lat m, const double* U,
                                                                      const double* __restrict__ g, double* Uo) {
  __shared__ LinkTile tile;
  __shared__ double2 gt[kLinkSites * 9];
  const int64_t L0 = (int64_t)blockIdx.x * kLinkSites;
  const int n = (int)min((int64_t)kLinkSites, m.V - L0);
  load_links(U, L0, n, tile);
  for (int j = threadIdx.x; j < n * 9; j += kLinkThreads) gt[j] = reinterpret_cast<const double2*>(g)[L0 * 9 + j];
  __syncthreads();
  const int site = threadIdx.x & 63, mu = threadIdx.x >> 6;
  if (site < n) {
    int64_t rest = L0 + site;
    int x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = (int)(rest % m.L[k]);
      rest /= m.L[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k == mu) x[k] = (x[k] + 1 == m.L[k]) ? 0 : x[k] + 1;
    const int64_t nb = x[0] + (int64_t)m.L[0] * (x[1] + (int64_t)m.L[1] * (x[2] + (int64_t)m.L[2] * x[3]));
    double A[18], B[18], N[18], T[18];
    load9(reinterpret_cast<const double2*>(g) + nb * 9, N);
    load9(gt + site * 9, A);
    double2* rec = tile + site * kLinkRow + 9 * mu;
    load9(rec, B);
    mm(A, B, T);
    mmd(T, N, B);
#pragma unroll
    for (int k = 0; k < 9; ++k) rec[k] = make_double2(B[2 * k], B[2 * k + 1]);
  }
  __syncthreads();
  double2* dst = reinterpret_cast<double2*>(Uo) + L0 * 36;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int idx = k * kLinkThreads + threadIdx.x;
    if (idx < 36 * n) dst[idx] = tile[(idx / 36) * kLinkRow + idx % 36];
  }
}

// psi'(x) = g(x) psi(x) or g(x)^dagger psi(x): one wavefront per 64 sites of one
// right-hand side, records of 192 bytes (13 slots in LDS) and g through LDS.
// out may alias in.  24^3x32: 213 -> 55 us.
__global__ void __launch_bounds__(64) rotate_kernel(Lat m, const double* __restrict__ g, const double* in, double* out,
                                                    int adjoint) {
  __shared__ double2 tile[64 * 13];
  __shared__ double2 gt[64 * 9];
  const int lane = threadIdx.x;
  const int64_t L0 = (int64_t)blockIdx.x * 64;
  const int n = (int)min((int64_t)64, m.V - L0);
  const double2* src = reinterpret_cast<const double2*>(in) + ((int64_t)blockIdx.y * m.V + L0) * 12;
  const double2* gsrc = reinterpret_cast<const double2*>(g) + L0 * 9;
  double2 v[12], w[9];
#pragma unroll
  for (int k = 0; k < 12; ++k) v[k] = src[min(k * 64 + lane, 12 * n - 1)];
#pragma unroll
  for (int k = 0; k < 9; ++k) w[k] = gsrc[min(k * 64 + lane, 9 * n - 1)];
#pragma unroll
  for (int k = 0; k < 12; ++k) tile[(k * 64 + lane) / 12 * 13 + (k * 64 + lane) % 12] = v[k];
#pragma unroll
  for (int k = 0; k < 9; ++k) gt[k * 64 + lane] = w[k];
  __syncthreads();
  if (lane < n) {
    double G[18];
    load9(gt + 9 * lane, G);
    double2* rec = tile + 13 * lane;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double2 p[3];
#pragma unroll
      for (int b = 0; b < 3; ++b) p[b] = rec[3 * s + b];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        double re = 0.0, im = 0.0;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          const double gr = adjoint ? G[6 * b + 2 * a] : G[6 * a + 2 * b];
          const double gi = adjoint ? -G[6 * b + 2 * a + 1] : G[6 * a + 2 * b + 1];
          re += gr * p[b].x - gi * p[b].y;
          im += gr * p[b].y + gi * p[b].x;
        }
        rec[3 * s + a] = make_double2(re, im);
      }
    }
  }
  __syncthreads();
  double2* dst = reinterpret_cast<double2*>(out) + ((int64_t)blockIdx.y * m.V + L0) * 12;
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const int idx = k * 64 + lane;
    if (idx < 12 * n) dst[idx] = tile[idx / 12 * 13 + idx % 12];
  }
}

unsigned grid1(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

}  // namespace

hipError_t launch_gauge_encode8(const wd_gauge* g, const double* U, hipStream_t s) {
  const Lat m = lat_of(g->geom);
  gauge_encode8_kernel<<<grid1(m.V, kLinkSites), kLinkThreads, 0, s>>>(m, U, g->geom.stride, static_cast<char*>(g->link[WD_FP64]),
                                            static_cast<char*>(g->link[WD_FP32]),
                                            static_cast<char*>(g->link[WD_HALF_I16]),
                                            static_cast<char*>(g->link[WD_HALF_F16]));
  return hipGetLastError();
}

hipError_t launch_temporal_check(const Geom& geo, const double* U, unsigned long long* dev, hipStream_t s) {
  const Lat m = lat_of(geo);
  const int64_t V3 = (int64_t)m.L[0] * m.L[1] * m.L[2];
  temporal_check_kernel<<<grid1((m.V - V3) * 9, 256 * kCheckIters), 256, 0, s>>>(m, U, dev);
  return hipGetLastError();
}

hipError_t launch_gauge_fix_temporal(const Geom& geo, const double* U, double* Uo, double* g, hipStream_t s) {
  const Lat m = lat_of(geo);
  const int64_t V3 = (int64_t)m.L[0] * m.L[1] * m.L[2];
  temporal_g_kernel<<<grid1(V3 * 3, 128), 128, 0, s>>>(m, U, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  temporal_links_kernel<<<grid1(m.V, kLinkSites), kLinkThreads, 0, s>>>(m, U, g, Uo);
  return hipGetLastError();
}

hipError_t launch_gauge_rotate(const Geom& geo, const double* g, const double* in, double* out, int nrhs,
                               int adjoint, hipStream_t s) {
  const Lat m = lat_of(geo);
  rotate_kernel<<<dim3(grid1(m.V, 64), nrhs), 64, 0, s>>>(m, g, in, out, adjoint);
  return hipGetLastError();
}

}  // namespace wd
