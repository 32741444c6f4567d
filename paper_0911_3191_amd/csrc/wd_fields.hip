// Conversions between the caller's canonical FP64 layouts and the device
// field formats: gauge links to 12-real rows (Appendix A.1) in each storage
// precision, spinors to site-coalesced chunk arrays with, for the 16-bit
// formats, a per-site norm (Section 4.6).
#include "wd_device.h"

namespace wd {

struct SiteMap {
  int L[4];
  int Lxh;
  int Vh;
};

// lex index of checkerboard site cb of parity p.
__device__ __forceinline__ int64_t lex_of(const SiteMap& m, int cb, int p) {
  int rest = cb / m.Lxh;
  const int xh = cb - rest * m.Lxh;
  const int y = rest % m.L[1];
  rest /= m.L[1];
  const int z = rest % m.L[2];
  const int t = rest / m.L[2];
  const int x = 2 * xh + ((p + y + z + t) & 1);
  return x + (int64_t)m.L[0] * (y + (int64_t)m.L[1] * (z + (int64_t)m.L[2] * t));
}

// Parity of lexicographic site L; its checkerboard index is L / 2 (Lx is even).
__device__ __forceinline__ int parity_of(const SiteMap& m, int L) {
  const int row = L / m.L[0];
  const int x = L - row * m.L[0];
  const int y = row % m.L[1];
  const int zt = row / m.L[1];
  const int z = zt % m.L[2];
  const int t = zt / m.L[2];
  return (x + y + z + t) & 1;
}

static SiteMap site_map(const Geom& g) {
  SiteMap m;
  for (int k = 0; k < 4; ++k) m.L[k] = g.L[k];
  m.Lxh = g.Lxh;
  m.Vh = g.Vh;
  return m;
}

// ---- gauge ------------------------------------------------------------------------
// One thread per (site, mu): rows a, b of U[lex][mu] into every precision of
// the mask.  16-bit: int16 q = rint(u * 32767) or binary16 u.
__global__ void __launch_bounds__(kLinkThreads) gauge_encode_kernel(SiteMap m, const double* __restrict__ U,
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
  const double2* rec = link_record(tile, mu, site);  // rows a, b are the first 12 reals
  double v[12];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    v[2 * k] = rec[k].x;
    v[2 * k + 1] = rec[k].y;
  }
  if (f64) {
#pragma unroll
    for (int k = 0; k < 6; ++k)
      reinterpret_cast<double2*>(const_cast<char*>(link_chunk<SF64>(f64, stride, par, mu, k)))[cb] =
          make_double2(v[2 * k], v[2 * k + 1]);
  }
  if (f32) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      reinterpret_cast<float4*>(const_cast<char*>(link_chunk<SF32>(f32, stride, par, mu, k)))[cb] =
          make_float4((float)v[4 * k], (float)v[4 * k + 1], (float)v[4 * k + 2], (float)v[4 * k + 3]);
  }
  if (i16) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      uint32_t w[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float a = fminf(fmaxf(rintf((float)v[4 * k + 2 * j] * 32767.0f), -32767.0f), 32767.0f);
        float b = fminf(fmaxf(rintf((float)v[4 * k + 2 * j + 1] * 32767.0f), -32767.0f), 32767.0f);
        w[j] = (uint32_t)(uint16_t)(int16_t)a | ((uint32_t)(uint16_t)(int16_t)b << 16);
      }
      reinterpret_cast<uint2*>(const_cast<char*>(link_chunk<SI16>(i16, stride, par, mu, k)))[cb] =
          make_uint2(w[0], w[1]);
    }
  }
  if (h16) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      uint32_t w[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        w[j] = (uint32_t)f_to_h16(pin_f32((float)v[4 * k + 2 * j])) |
               ((uint32_t)f_to_h16(pin_f32((float)v[4 * k + 2 * j + 1])) << 16);
      reinterpret_cast<uint2*>(const_cast<char*>(link_chunk<SF16>(h16, stride, par, mu, k)))[cb] =
          make_uint2(w[0], w[1]);
    }
  }
}

hipError_t launch_gauge_encode(const wd_gauge* g, const double* U, hipStream_t s) {
  SiteMap m = site_map(g->geom);
  gauge_encode_kernel<<<(2 * m.Vh + kLinkSites - 1) / kLinkSites, kLinkThreads, 0, s>>>(
      m, U, g->geom.stride, static_cast<char*>(g->link[WD_FP64]), static_cast<char*>(g->link[WD_FP32]),
      static_cast<char*>(g->link[WD_HALF_I16]), static_cast<char*>(g->link[WD_HALF_F16]));
  return hipGetLastError();
}

// ---- spinors ----------------------------------------------------------------------
// Change of spin basis in FP64 (Appendix B), v = [spin][colour][re, im]:
// to_uk: v <- S v with S = [[0, 1, 0, 1], [-1, 0, -1, 0], [0, 1, 0, -1],
// [-1, 0, 1, 0]] / sqrt(2) (DeGrand-Rossi to UKQCD); otherwise v <- S^T v.
__device__ __forceinline__ void change_basis(double (&v)[24], bool to_uk) {
  constexpr double r = 0.70710678118654752440;  // 1 / sqrt(2)
#pragma unroll
  for (int k = 0; k < 6; ++k) {  // colour and re / im
    const double a0 = v[k], a1 = v[6 + k], a2 = v[12 + k], a3 = v[18 + k];
    if (to_uk) {
      v[k] = r * (a1 + a3);
      v[6 + k] = -r * (a0 + a2);
      v[12 + k] = r * (a1 - a3);
      v[18 + k] = r * (a2 - a0);
    } else {
      v[k] = -r * (a1 + a3);
      v[6 + k] = r * (a0 + a2);
      v[12 + k] = r * (a3 - a1);
      v[18 + k] = r * (a0 - a2);
    }
  }
}

// Per-RHS factor of the solver's unit-source scaling: 1 / |b| (scale = 1) or
// |b| (scale = 2) from the solver scalars sc; 1 without scaling or when |b|
// is zero or not finite.
__device__ __forceinline__ double bnorm_factor(const double* __restrict__ sc, int scale, int r) {
  if (!scale) return 1.0;
  const double bn = sc[r * SC_COUNT + SC_BNORM];
  if (!(bn > 0.0) || !isfinite(bn)) return 1.0;
  return scale == 1 ? 1.0 / bn : bn;
}

// One site: 24 canonical reals (DeGrand-Rossi basis) into the field in
// `basis`, times bnorm_factor after the change of basis when scale is set.
template <class S>
__device__ __forceinline__ void encode_site(FieldView f, int r, int cb, const double* __restrict__ src, int basis,
                                            const double* __restrict__ sc, int scale) {
  using R = typename S::real;
  double v[24];
#pragma unroll
  for (int n = 0; n < 24; ++n) v[n] = src[n];
  if (basis == kBasisUK) change_basis(v, true);
  if (scale) {
    const double k = bnorm_factor(sc, scale, r);
#pragma unroll
    for (int n = 0; n < 24; ++n) v[n] = k * v[n];
  }
  Spinor<R> s;
#pragma unroll
  for (int n = 0; n < 12; ++n) s.v[n / 3][n % 3] = {static_cast<R>(v[2 * n]), static_cast<R>(v[2 * n + 1])};
  store_spinor<S>(f, r, cb, s);
}

// One site back: the field's values, times bnorm_factor before the change of
// basis when scale is set, into 24 canonical reals.
template <class S>
__device__ __forceinline__ void decode_site(FieldView f, int r, int cb, double* __restrict__ dst, int basis,
                                            const double* __restrict__ sc, int scale) {
  using R = typename S::real;
  Spinor<R> s;
  load_spinor<S>(f, r, cb, s);
  double v[24];
#pragma unroll
  for (int n = 0; n < 12; ++n) {
    v[2 * n] = static_cast<double>(s.v[n / 3][n % 3].re);
    v[2 * n + 1] = static_cast<double>(s.v[n / 3][n % 3].im);
  }
  if (scale) {
    const double k = bnorm_factor(sc, scale, r);
#pragma unroll
    for (int n = 0; n < 24; ++n) v[n] = k * v[n];
  }
  if (basis == kBasisUK) change_basis(v, false);
#pragma unroll
  for (int n = 0; n < 24; ++n) dst[n] = v[n];
}

// The canonical records (192 bytes a site) pass through LDS, so that they are
// moved 16 bytes a lane in address order: one thread per record touches 64
// lines with each instruction, which cost most in the decode (stores of 16
// bytes each, 192 bytes apart).  A wavefront owns the 64 sites of its lanes
// and needs no other one; a record takes 13 slots of 16 bytes in the tile,
// which spreads the lanes' own reads and writes over all banks.  Per pass
// over a binary16 field at 48^3x96, 12 right-hand sides: encode 3.08 -> 2.89 ms,
// decode 3.71 -> 2.79 ms; at 24^3x32, one: 10.6 -> 10.3 and 18.9 -> 11.2 us.
constexpr int kTileSites = 64;  // sites per workgroup, one wavefront
constexpr int kTileRow = 13;    // 16-byte slots per record: 12 and one of padding

// Moves the records of n consecutive lanes' sites between the canonical array
// and the tile; rec: this lane's record number (CONTIG: those of the lanes
// follow one another).  The stores are marked streaming, so that the fields keep
// the caches (24^3x32 binary16 decode 11.2 -> 10 us).  It holds for a caller who
// feeds the output to the next call too: wilson_mat_pc applied again and again,
// plain / streaming in microseconds, 8^4 FP64 14.5 / 14.4, 20x14x10x18 int16 with
// 5 right-hand sides 36.5 / 36.5, binary16 24^3x32 54.2 / 54.4, 32^4 112.3 / 110.5,
// 24^3x32 with 4 (170 MB of records) 161 / 154, 48^3x96 (1.02 GB) 1183 / 1149.
template <bool CONTIG, bool STORE>
__device__ __forceinline__ void move_records(double2* __restrict__ canon, double2* __restrict__ tile, int rec, int n) {
  const int lane = threadIdx.x;
  const int64_t first = __builtin_amdgcn_readfirstlane(rec);
  double2 v[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const int idx = k * kTileSites + lane;
    const int site = idx / 12, part = idx - 12 * site;
    if constexpr (STORE) v[k] = tile[kTileRow * site + part];
    // loads without a branch, all in flight together: past the end they repeat the last piece
    else if constexpr (CONTIG) v[k] = canon[first * 12 + min(idx, 12 * n - 1)];
    else v[k] = canon[(int64_t)__shfl(rec, site) * 12 + part];
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const int idx = k * kTileSites + lane;
    const int site = idx / 12, part = idx - 12 * site;
    if constexpr (!STORE) {
      tile[kTileRow * site + part] = v[k];
    } else {
      const int64_t at = CONTIG ? first * 12 + idx : (int64_t)__shfl(rec, site) * 12 + part;
      if (site < n) st16<true>(reinterpret_cast<dvec2*>(canon) + at, dvec2{v[k].x, v[k].y});
    }
  }
}

// FULL = false: canonical array is a parity array [nrhs][Vh][24]; FULL = true:
// it is a full lattice [nrhs][V][24] and the field holds its sites of parity
// `parity`.  The canonical array is in the DeGrand-Rossi basis, the field in
// `basis`.
template <class S, bool FULL>
__global__ void __launch_bounds__(kTileSites) spinor_encode_kernel(SiteMap m, FieldView f,
                                                                   const double* __restrict__ canon, int parity,
                                                                   int basis, const double* __restrict__ sc,
                                                                   int scale) {
  __shared__ double2 tile[kTileSites * kTileRow];
  const int cb = blockIdx.x * kTileSites + threadIdx.x;
  const int r = blockIdx.y;
  const int n = min(kTileSites, m.Vh - (int)blockIdx.x * kTileSites);
  const double* src = canon + (int64_t)r * (FULL ? 2 : 1) * m.Vh * 24;
  const int rec = FULL ? (int)lex_of(m, min(cb, m.Vh - 1), parity) : cb;
  move_records<!FULL, false>(reinterpret_cast<double2*>(const_cast<double*>(src)), tile, rec, n);
  __syncthreads();
  if ((int)threadIdx.x >= n) return;
  encode_site<S>(f, r, cb, reinterpret_cast<const double*>(tile + kTileRow * threadIdx.x), basis, sc, scale);
}

template <class S, bool FULL>
__global__ void __launch_bounds__(kTileSites) spinor_decode_kernel(SiteMap m, FieldView f, double* __restrict__ canon,
                                                                   int parity, int basis,
                                                                   const double* __restrict__ sc, int scale) {
  __shared__ double2 tile[kTileSites * kTileRow];
  const int cb = blockIdx.x * kTileSites + threadIdx.x;
  const int r = blockIdx.y;
  const int n = min(kTileSites, m.Vh - (int)blockIdx.x * kTileSites);
  if ((int)threadIdx.x < n)
    decode_site<S>(f, r, cb, reinterpret_cast<double*>(tile + kTileRow * threadIdx.x), basis, sc, scale);
  __syncthreads();
  double* dst = canon + (int64_t)r * (FULL ? 2 : 1) * m.Vh * 24;
  const int rec = FULL ? (int)lex_of(m, min(cb, m.Vh - 1), parity) : cb;
  move_records<!FULL, true>(reinterpret_cast<double2*>(dst), tile, rec, n);
}

// Both parities of a canonical full lattice [nrhs][V][24] (FP64 fields) in one
// pass: a workgroup takes 64 consecutive lexicographic sites, whose records
// form one contiguous block; lane k works on site L0 + k, whose even / odd
// sites come from (go to) fe / fo.
__global__ void __launch_bounds__(kTileSites) spinor_encode_both_kernel(SiteMap m, FieldView fe, FieldView fo,
                                                                        const double* __restrict__ canon,
                                                                        int basis, const double* __restrict__ sc,
                                                                        int scale) {
  __shared__ double2 tile[kTileSites * kTileRow];
  const int L = blockIdx.x * kTileSites + threadIdx.x;
  const int r = blockIdx.y;
  const int n = min(kTileSites, 2 * m.Vh - (int)blockIdx.x * kTileSites);  // sites in this block
  const double* src = canon + (int64_t)r * 2 * m.Vh * 24;
  move_records<true, false>(reinterpret_cast<double2*>(const_cast<double*>(src)), tile, L, n);
  __syncthreads();
  if ((int)threadIdx.x >= n) return;
  encode_site<SF64>(parity_of(m, L) ? fo : fe, r, L >> 1,
                    reinterpret_cast<const double*>(tile + kTileRow * threadIdx.x), basis, sc, scale);
}

__global__ void __launch_bounds__(kTileSites) spinor_decode_both_kernel(SiteMap m, FieldView fe, FieldView fo,
                                                                        double* __restrict__ canon, int basis,
                                                                        const double* __restrict__ sc, int scale) {
  __shared__ double2 tile[kTileSites * kTileRow];
  const int L = blockIdx.x * kTileSites + threadIdx.x;
  const int r = blockIdx.y;
  const int n = min(kTileSites, 2 * m.Vh - (int)blockIdx.x * kTileSites);
  if ((int)threadIdx.x < n)
    decode_site<SF64>(parity_of(m, L) ? fo : fe, r, L >> 1, reinterpret_cast<double*>(tile + kTileRow * threadIdx.x),
                      basis, sc, scale);
  __syncthreads();
  move_records<true, true>(reinterpret_cast<double2*>(canon + (int64_t)r * 2 * m.Vh * 24), tile, L, n);
}

template <class S>
static hipError_t enc_typed(const Geom& g, Field f, const double* canon, int full_parity, int basis,
                            const double* sc, int scale, hipStream_t s) {
  dim3 grid((g.Vh + kTileSites - 1) / kTileSites, f.nrhs);
  const FieldView v{f.ptr, f.stride, f.nrhs};
  if (full_parity < 0)
    spinor_encode_kernel<S, false><<<grid, kTileSites, 0, s>>>(site_map(g), v, canon, 0, basis, sc, scale);
  else
    spinor_encode_kernel<S, true><<<grid, kTileSites, 0, s>>>(site_map(g), v, canon, full_parity, basis, sc, scale);
  return hipGetLastError();
}

template <class S>
static hipError_t dec_typed(const Geom& g, double* canon, Field f, int full_parity, int basis,
                            const double* sc, int scale, hipStream_t s) {
  dim3 grid((g.Vh + kTileSites - 1) / kTileSites, f.nrhs);
  const FieldView v{f.ptr, f.stride, f.nrhs};
  if (full_parity < 0)
    spinor_decode_kernel<S, false><<<grid, kTileSites, 0, s>>>(site_map(g), v, canon, 0, basis, sc, scale);
  else
    spinor_decode_kernel<S, true><<<grid, kTileSites, 0, s>>>(site_map(g), v, canon, full_parity, basis, sc, scale);
  return hipGetLastError();
}

hipError_t launch_spinor_encode_map(const Geom& g, wd_prec p, Field f, const double* canon,
                                    int full_parity, hipStream_t s, int basis, const double* sc,
                                    int scale) {
  if (basis != kBasisDR && basis != kBasisUK) return hipErrorInvalidValue;
  if (scale < 0 || scale > 2 || (scale && !sc)) return hipErrorInvalidValue;
  switch (p) {
    case WD_FP64: return enc_typed<SF64>(g, f, canon, full_parity, basis, sc, scale, s);
    case WD_FP32: return enc_typed<SF32>(g, f, canon, full_parity, basis, sc, scale, s);
    case WD_HALF_I16: return enc_typed<SI16>(g, f, canon, full_parity, basis, sc, scale, s);
    case WD_HALF_F16: return enc_typed<SF16>(g, f, canon, full_parity, basis, sc, scale, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_spinor_decode_map(const Geom& g, wd_prec p, double* canon, Field f,
                                    int full_parity, hipStream_t s, int basis, const double* sc,
                                    int scale) {
  if (basis != kBasisDR && basis != kBasisUK) return hipErrorInvalidValue;
  if (scale < 0 || scale > 2 || (scale && !sc)) return hipErrorInvalidValue;
  switch (p) {
    case WD_FP64: return dec_typed<SF64>(g, canon, f, full_parity, basis, sc, scale, s);
    case WD_FP32: return dec_typed<SF32>(g, canon, f, full_parity, basis, sc, scale, s);
    case WD_HALF_I16: return dec_typed<SI16>(g, canon, f, full_parity, basis, sc, scale, s);
    case WD_HALF_F16: return dec_typed<SF16>(g, canon, f, full_parity, basis, sc, scale, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_spinor_encode_both(const Geom& g, Field fe, Field fo, const double* canon, hipStream_t s,
                                     int basis, const double* sc, int scale) {
  if (basis != kBasisDR && basis != kBasisUK) return hipErrorInvalidValue;
  if (scale < 0 || scale > 2 || (scale && !sc) || fe.nrhs != fo.nrhs) return hipErrorInvalidValue;
  dim3 grid((unsigned)((2 * (int64_t)g.Vh + kTileSites - 1) / kTileSites), fe.nrhs);
  spinor_encode_both_kernel<<<grid, kTileSites, 0, s>>>(site_map(g), FieldView{fe.ptr, fe.stride, fe.nrhs},
                                                        FieldView{fo.ptr, fo.stride, fo.nrhs}, canon, basis, sc,
                                                        scale);
  return hipGetLastError();
}

hipError_t launch_spinor_decode_both(const Geom& g, double* canon, Field fe, Field fo, hipStream_t s,
                                     int basis, const double* sc, int scale) {
  if (basis != kBasisDR && basis != kBasisUK) return hipErrorInvalidValue;
  if (scale < 0 || scale > 2 || (scale && !sc) || fe.nrhs != fo.nrhs) return hipErrorInvalidValue;
  dim3 grid((unsigned)((2 * (int64_t)g.Vh + kTileSites - 1) / kTileSites), fe.nrhs);
  spinor_decode_both_kernel<<<grid, kTileSites, 0, s>>>(site_map(g), FieldView{fe.ptr, fe.stride, fe.nrhs},
                                                        FieldView{fo.ptr, fo.stride, fo.nrhs}, canon, basis, sc,
                                                        scale);
  return hipGetLastError();
}

hipError_t launch_spinor_encode(const Geom& g, wd_prec p, Field f, const double* canon,
                                hipStream_t s, int basis) {
  return launch_spinor_encode_map(g, p, f, canon, -1, s, basis);
}

hipError_t launch_spinor_decode(const Geom& g, wd_prec p, double* canon, Field f, hipStream_t s,
                                int basis) {
  return launch_spinor_decode_map(g, p, canon, f, -1, s, basis);
}

}  // namespace wd
