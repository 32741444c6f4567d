// Dslash with one wavefront per hop, for launches too small to fill the chip
// with one thread per output site.
//
// A workgroup of eight wavefronts owns 64 output sites of one right-hand
// side.  Wavefront h computes hop h of all of them (h / 2: direction, h odd:
// backward): it gathers its link and its neighbour and forms the product of
// the link and the projected half spinor, U h, which it leaves in LDS.  The
// first wavefront then accumulates the eight products in the order of the
// one-thread kernels, with the same fused multiply-adds, and finishes the
// site, so the results are the same bits.
//
// What bounds a small launch is latency: the one-thread kernels walk the four
// directions one after the other, each waiting for its own loads, with few
// wavefronts per SIMD to hide them.  Here all eight hops of a site are in
// flight at once.  Measured per launch (UKQCD basis, D, in a hipGraph; best
// one-thread shape -> this kernel, microseconds): 8^4 binary16 5.7 -> 3.9,
// FP64 6.8 -> 4.9; 16^3x32 FP32 13.7 -> 9.0; 24^3x32 binary16 18.8 -> 15.5,
// FP32 30.7 -> 21.5, FP64 60.8 -> 45.3; 32^3x32 binary16 36.2 -> 29.1.  Past
// the cache the fewer, longer wavefronts of the one-thread kernels win (32^3x64
// binary16 64 against 71): split_pays in wd_tune.cpp has the line.  FP64
// launches of more than 65,536 site right-hand sides give each wavefront both
// hops of a direction (20x14x10x18 with 12 right-hand sides 46 -> 41, 24^3x32
// 46.4 -> 45.3; at 8^4 4.9 -> 5.3, so the smallest keep one).
#pragma once

#include "wd_dslash_impl.h"

namespace wd {

constexpr int kSplitSites = 64;  // sites per workgroup, one wavefront's lanes

// Product of hop (MU, BACK): w = U h (forward) or U^dagger h (backward) of
// the projected neighbour, and the factor that its accumulation applies.
template <class S, int MU, bool BACK, bool DAGGER, int RECON, int BASIS>
__device__ __forceinline__ void hop_product(const DslashGeom& g, const char* __restrict__ links,
                                            const SpinorBuf<S>& in, int p, int cb, const HopIdx& hi, float one,
                                            cx<typename S::real> (&w)[2][3], typename S::real& scale) {
  using R = typename S::real;
  using G = GammaB<MU, BASIS>;
  constexpr int sh = (BACK == DAGGER) ? 2 : 0;  // forward hops carry 1 - gamma, backward 1 + gamma; the adjoint swaps
  constexpr bool HALF = MU == 3 && BASIS == kBasisUK;
  constexpr int BASE = (BACK == DAGGER) ? 2 : 0;  // spins that a temporal projector keeps
  const int nb = BACK ? hi.nb : hi.nf;
  const bool flip = BACK ? hi.flip_b : hi.flip_f;
  const bool unit = BACK ? hi.unit_b : hi.unit_f;
  const int lpar = BACK ? 1 - p : p, lsite = BACK ? nb : cb;
  if constexpr (S::prec == WD_HALF_F16) {
    Link16 U;
    link_of16<S, RECON, 0>(g, links, lpar, MU, lsite, unit, U);
    float sc;
    uint32_t f1[2][3], f2[2][3];
    if constexpr (HALF) {
      uint32_t h[6];
      gather_half16w<BASE>(in, nb, h, sc);
      sc = 2.0f * sc;
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          f1[k][c] = BACK ? h[3 * k + c] : wconj(h[3 * k + c]);
          f2[k][c] = BACK ? wmi(h[3 * k + c]) : wswap(h[3 * k + c]);
        }
    } else {
      constexpr int F1 = BACK ? kFormId : kFormConj, F2 = BACK ? kFormMi : kFormSwap;
      Raw16 psi;
      gather_spinor16<S>(in, nb, psi, sc);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const uint32_t a0 = psi.w[c], b0 = psi.w[3 * (2 + G::P0) + c];
        const uint32_t a1 = psi.w[3 + c], b1 = psi.w[3 * (2 + G::P1) + c];
        f1[0][c] = pk_form<F1, G::PH0 + sh>(a0, b0);
        f2[0][c] = pk_form<F2, G::PH0 + sh>(a0, b0);
        f1[1][c] = pk_form<F1, G::PH1 + sh>(a1, b1);
        f2[1][c] = pk_form<F2, G::PH1 + sh>(a1, b1);
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int a = 0; a < 3; ++a) w[k][a] = su3_row16<BACK>(U, a, f1[k], f2[k]);
    scale = flip ? -sc : sc;
  } else {
    Link<R> U;
    if (unit) unit_link(U);
    else gather_link<S, RECON, 0>(g, links, lpar, MU, lsite, U);
    cx<R> h[2][3];
    R sc = R(1);
    if constexpr (HALF) {
      if constexpr (kHalf<S>) {
        float s16;
        gather_half16<S, BASE>(in, nb, h, s16);
        sc = 2.0f * s16;
      } else {
        gather_half<S, BASE>(in, nb, h);
        sc = R(2);
      }
    } else if constexpr (kHalf<S>) {
      Raw16 psi;
      gather_spinor16<S>(in, nb, psi, sc);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        h[0][c] = proj16<G::PH0 + sh, S>(psi.w[c], psi.w[3 * (2 + G::P0) + c], one);
        h[1][c] = proj16<G::PH1 + sh, S>(psi.w[3 + c], psi.w[3 * (2 + G::P1) + c], one);
      }
    } else {
      Spinor<R> psi;
      gather_spinor<S>(in, nb, psi);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        h[0][c] = psi.v[0][c] + iph<G::PH0 + sh>(psi.v[2 + G::P0][c]);
        h[1][c] = psi.v[1][c] + iph<G::PH1 + sh>(psi.v[2 + G::P1][c]);
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        cx<R> z = {R(0), R(0)};
        if constexpr (!BACK) {
          z = cmac(z, U.u[a][0], h[k][0]);
          z = cmac(z, U.u[a][1], h[k][1]);
          z = cmac(z, U.u[a][2], h[k][2]);
        } else {
          z = cmacc(z, U.u[0][a], h[k][0]);
          z = cmacc(z, U.u[1][a], h[k][1]);
          z = cmacc(z, U.u[2][a], h[k][2]);
        }
        w[k][a] = z;
      }
    scale = flip ? -sc : sc;
  }
}

// What a hop left in LDS for this lane's site.
template <typename R>
struct HopVals {
  R w[12], sc;
};
template <typename R>
__device__ __forceinline__ HopVals<R> hop_vals(const R (&wbuf)[8][12][kSplitSites], const R (&sbuf)[8][kSplitSites],
                                               int slot, int lane) {
  HopVals<R> q;
#pragma unroll
  for (int k = 0; k < 12; ++k) q.w[k] = wbuf[slot][k][lane];
  q.sc = sbuf[slot][lane];
  return q;
}

// acc += scale * (1 -+ gamma) expansion of w, one fused multiply-add per real
// (mul_acc / mul_acc_half of the one-thread kernels).
template <int MU, bool BACK, bool DAGGER, int BASIS, typename R>
__device__ __forceinline__ void hop_accumulate(Spinor<R>& acc, const HopVals<R>& q) {
  using G = GammaB<MU, BASIS>;
  constexpr int sh = (BACK == DAGGER) ? 2 : 0;
  constexpr int BASE = (BACK == DAGGER) ? 2 : 0;
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const cx<R> z = {q.w[6 * k + 2 * a], q.w[6 * k + 2 * a + 1]};
      const R scale = q.sc;
      if constexpr (MU == 3 && BASIS == kBasisUK) {
        cx<R>& t = acc.v[BASE + k][a];
        t = {fmar(scale, z.re, t.re), fmar(scale, z.im, t.im)};
      } else {
        cx<R>& u = acc.v[k][a];
        u = {fmar(scale, z.re, u.re), fmar(scale, z.im, u.im)};
        cx<R>& l = acc.v[2 + (k == 0 ? G::P0 : G::P1)][a];
        const cx<R> zl = (k == 0) ? iph<sh - G::PH0 + 4>(z) : iph<sh - G::PH1 + 4>(z);
        l = {fmar(scale, zl.re, l.re), fmar(scale, zl.im, l.im)};
      }
    }
}

// Packed contents of one site of a field, decoded later: fewer registers
// than the decoded spinor while it waits.
template <class S>
struct RawSite {
  uint4 c[S::NCH];
  float nm;
};
template <class S>
__device__ __forceinline__ void load_raw(const FieldView& f, int r, int64_t i, RawSite<S>& q) {
  if constexpr (kHalf<S>) q.nm = norm_base(f, r)[i];
#pragma unroll
  for (int k = 0; k < S::NCH; ++k) q.c[k] = reinterpret_cast<const uint4*>(chunk_base<S>(f, r, k))[i];
}
// The values of load_spinor.
template <class S>
__device__ __forceinline__ void decode_raw(const RawSite<S>& q, Spinor<typename S::real>& s) {
  if constexpr (S::prec == WD_FP64) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const double2 c = __builtin_bit_cast(double2, q.c[k]);
      s.v[k / 3][k % 3] = {c.x, c.y};
    }
  } else if constexpr (S::prec == WD_FP32) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const float4 c = __builtin_bit_cast(float4, q.c[k]);
      s.v[(2 * k) / 3][(2 * k) % 3] = {c.x, c.y};
      s.v[(2 * k + 1) / 3][(2 * k + 1) % 3] = {c.z, c.w};
    }
  } else {
    const float sc = (S::prec == WD_HALF_I16) ? q.nm / 32767.0f : q.nm;
#pragma unroll
    for (int n = 0; n < 12; ++n) {
      const uint4 c = q.c[n / 4];
      const uint32_t w = n % 4 == 0 ? c.x : n % 4 == 1 ? c.y : n % 4 == 2 ? c.z : c.w;
      const uint16_t lo = (uint16_t)(w & 0xffffu), hi = (uint16_t)(w >> 16);
      if constexpr (S::prec == WD_HALF_I16) s.v[n / 3][n % 3] = {(float)(int16_t)lo * sc, (float)(int16_t)hi * sc};
      else s.v[n / 3][n % 3] = {h16_to_f(lo) * sc, h16_to_f(hi) * sc};
    }
  }
}

// Wavefronts per SIMD that the register count has to allow: three workgroups
// per CU (FP64 with one hop per wavefront: two).  The FP64 sums of DOT_OX take
// more registers: FP32 spills 68 at six and takes two workgroups (6 spilled; a
// 24^3x32 solve 8.4 ms); the 16-bit formats spill 20 and are still faster
// with three (6.2 ms instead of 6.4 with none spilled).
template <class S, int HPW, int DOT>
constexpr int split_waves() {
  if (S::prec == WD_FP64) return HPW == 2 ? 3 : 4;
  return S::prec == WD_FP32 && DOT == DOT_OX ? 4 : 6;
}

// HPW: hops per wavefront (2: both of one direction, four wavefronts).
template <class S, bool DAGGER, bool XPAY, int DOT, int RECON, int BASIS, int HPW, class S2 = S>
__global__ void __launch_bounds__(512 / HPW, (split_waves<S, HPW, DOT>())) dslash_split_kernel(DslashGeom g, const char* __restrict__ links,
                                                                  FieldView out, FieldView in, FieldView xs,
                                                                  FieldView ys, typename S::real a, int p,
                                                                  const int* __restrict__ sel,
                                                                  double* __restrict__ partials, EncView enc) {
  using R = typename S::real;
  __shared__ R wbuf[8][12][kSplitSites];
  __shared__ R sbuf[8][kSplitSites];
  const int lane = threadIdx.x & 63;
  const int hop = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // ---- which 64 sites and which RHS this workgroup owns (mapping of dslash_kernel, one sub-slab) ----
  const int xcd = blockIdx.x & 7;
  const int j = blockIdx.x >> 3;
  int site_block, group, pid, cb, xh, X1, X2, X3;
  bool valid;
  if (g.slab) {
    site_block = j / g.ngroups;
    group = j - site_block * g.ngroups;
    if (site_block >= g.site_blocks) return;
    pid = xcd * g.site_blocks + site_block;
    const int s_raw = site_block * kSplitSites + lane;
    valid = s_raw < (g.Vh >> 3);
    const int s_local = valid ? s_raw : (g.Vh >> 3) - 1;
    X3 = (int)fdiv((uint32_t)s_local, g.div_sub_t);
    const int r2 = s_local - X3 * g.sub_t_sites;
    const int zl = (int)fdiv((uint32_t)r2, g.div_sub_plane);
    const int r3 = r2 - zl * g.sub_plane;
    X1 = (int)fdiv((uint32_t)r3, g.div_lxh);
    xh = r3 - X1 * g.Lxh;
    X2 = xcd * (g.L[2] >> 3) + zl;
    cb = xh + g.Lxh * (X1 + g.L[1] * (X2 + g.L[2] * X3));
  } else {
    const int per = (g.site_blocks * g.ngroups + 7) >> 3;
    const int L = xcd * per + j;
    if (j >= per || L >= g.site_blocks * g.ngroups) return;
    site_block = L / g.ngroups;
    group = L - site_block * g.ngroups;
    pid = site_block;
    cb = site_block * kSplitSites + lane;
    valid = cb < g.Vh;
    if (!valid) cb = g.Vh - 1;  // works on the last site and stores nothing
    const int row = (int)fdiv((uint32_t)cb, g.div_lxh);
    xh = cb - row * g.Lxh;
    const int zt = (int)fdiv((uint32_t)row, g.div_ly);
    X1 = row - zt * g.L[1];
    X3 = (int)fdiv((uint32_t)zt, g.div_lz);
    X2 = zt - X3 * g.L[2];
  }
  int r = group;
  if (g.mapped) r = sel[group];
  else if (sel && !sel[group]) return;

  const int row = X1 + g.L[1] * (X2 + g.L[2] * X3);
  const int X[4] = {2 * xh + ((p + X1 + X2 + X3) & 1), X1, X2, X3};
  const float one = pin_f32(1.0f);  // see proj16
  const SpinorBuf<S> ib = spinor_buf<S>(in, r);
  auto leave = [&](int slot, const cx<R>(&w)[2][3], R sc) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        wbuf[slot][6 * k + 2 * c][lane] = w[k][c].re;
        wbuf[slot][6 * k + 2 * c + 1][lane] = w[k][c].im;
      }
    sbuf[slot][lane] = sc;
  };
  cx<R> w[2][3];
  R sc;
  if constexpr (HPW == 2) {
    cx<R> v[2][3];
    R sv;
#define WD_DIR(MU)                                                                                               \
  {                                                                                                              \
    const HopIdx hi = hop_index<MU>(g, xh, row, X);                                                              \
    hop_product<S, MU, false, DAGGER, RECON, BASIS>(g, links, ib, p, cb, hi, one, w, sc);                        \
    hop_product<S, MU, true, DAGGER, RECON, BASIS>(g, links, ib, p, cb, hi, one, v, sv);                         \
  }
    if (hop == 0) WD_DIR(0)
    else if (hop == 1) WD_DIR(1)
    else if (hop == 2) WD_DIR(2)
    else WD_DIR(3)
#undef WD_DIR
    leave(2 * hop, w, sc);
    leave(2 * hop + 1, v, sv);
  } else {
#define WD_HOP(MU, BACK) \
  hop_product<S, MU, BACK, DAGGER, RECON, BASIS>(g, links, ib, p, cb, hop_index<MU>(g, xh, row, X), one, w, sc)
    switch (hop) {
      case 0: WD_HOP(0, false); break;
      case 1: WD_HOP(0, true); break;
      case 2: WD_HOP(1, false); break;
      case 3: WD_HOP(1, true); break;
      case 4: WD_HOP(2, false); break;
      case 5: WD_HOP(2, true); break;
      case 6: WD_HOP(3, false); break;
      default: WD_HOP(3, true);
    }
#undef WD_HOP
    leave(hop, w, sc);
  }
  // the finishing wavefront's x and y loads are in flight across the barrier
  // (FP64: only x, the registers of both would cost a workgroup per CU)
  constexpr bool NEEDS_Y = DOT == DOT_YO || (DOT == DOT_OX && S::prec != WD_FP64) || DOT == DOT_RES || DOT == DOT_RES_ENC;
  RawSite<S> xr, yr;
  if (hop == 0) {
    if constexpr (XPAY) load_raw<S>(xs, r, cb, xr);
    if constexpr (NEEDS_Y && S::prec != WD_FP64) load_raw<S>(ys, r, cb, yr);
  }
  __syncthreads();
  if (hop != 0) return;
  // a fence after each hop keeps the LDS reads of all of them from piling up in
  // registers; without a dot (AHEAD) there is room for the next hop's reads
  // beside this one's arithmetic
  constexpr bool AHEAD = DOT == DOT_NONE && !XPAY && S::prec != WD_FP64;
  Spinor<R> acc[1];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[0].v[s][c] = {R(0), R(0)};
  HopVals<R> q = hop_vals<R>(wbuf, sbuf, 0, lane), qn;
#define WD_ACC(MU, BACK, SLOT)                                                      \
  if constexpr (AHEAD && SLOT < 7) qn = hop_vals<R>(wbuf, sbuf, SLOT + 1, lane);    \
  hop_accumulate<MU, BACK, DAGGER, BASIS>(acc[0], q);                               \
  hop_fence<R, 1>(acc);                                                             \
  if constexpr (SLOT < 7) q = AHEAD ? qn : hop_vals<R>(wbuf, sbuf, SLOT + 1, lane)
  WD_ACC(0, false, 0);
  WD_ACC(0, true, 1);
  WD_ACC(1, false, 2);
  WD_ACC(1, true, 3);
  WD_ACC(2, false, 4);
  WD_ACC(2, true, 5);
  WD_ACC(3, false, 6);
  WD_ACC(3, true, 7);
#undef WD_ACC
  Spinor<R> x, y;
  if constexpr (XPAY) decode_raw<S>(xr, x);
  if constexpr (NEEDS_Y) {
    if constexpr (S::prec == WD_FP64) load_spinor<S>(ys, r, cb, y);
    else decode_raw<S>(yr, y);
  }
  finish_rhs<S, XPAY, DOT, S2, true>(g, acc[0], r, cb, valid, pid, out, xs, ys, a, partials, enc, &x, &y);
}

// Geometry of a split launch: workgroups of 64 sites, four to each 256-site
// record of the one-thread kernels (missing ones at the end write zeros).
static DslashGeom make_split_geom(const Geom& geo, int nrhs, const LaunchCfg& c) {
  LaunchCfg one{1, 256};
  one.out_nt = c.out_nt;
  DslashGeom g = make_dgeom(geo, nrhs, one);
  g.site_blocks *= 256 / kSplitSites;
  return g;
}

template <class S, bool DAGGER, bool XPAY, int RECON, int BASIS, int HPW>
static void launch_split_dot(int dot, unsigned grid, hipStream_t s, const DslashGeom& g, const char* links,
                             FieldView fo, FieldView fi, FieldView fx, FieldView fy, typename S::real a, int p,
                             const int* sel, double* partials, EncView enc, wd_prec enc_prec) {
  constexpr bool UK = BASIS == kBasisUK, D64 = S::prec == WD_FP64;
#define WD_SPLIT(DOTMODE, S2)                                                                     \
  dslash_split_kernel<S, DAGGER, XPAY, DOTMODE, RECON, BASIS, HPW, S2><<<grid, 512 / HPW, 0, s>>>(  \
      g, links, fo, fi, fx, fy, a, p, sel, partials, enc)
  if constexpr (UK && XPAY && !DAGGER) {
    if (dot == DOT_YO) return (void)WD_SPLIT(DOT_YO, S);
    if (dot == DOT_OX) return (void)WD_SPLIT(DOT_OX, S);
    if (dot == DOT_OO) return (void)WD_SPLIT(DOT_OO, S);
    if constexpr (D64) {
      if (dot == DOT_RES) return (void)WD_SPLIT(DOT_RES, S);
      if (dot == DOT_RES_ENC && enc_prec == WD_FP32) return (void)WD_SPLIT(DOT_RES_ENC, SF32);
      if (dot == DOT_RES_ENC && enc_prec == WD_HALF_I16) return (void)WD_SPLIT(DOT_RES_ENC, SI16);
      if (dot == DOT_RES_ENC) return (void)WD_SPLIT(DOT_RES_ENC, SF16);
    }
  }
  if constexpr (UK && XPAY && DAGGER && D64) {
    if (dot == DOT_ENC && enc_prec == WD_FP32) return (void)WD_SPLIT(DOT_ENC, SF32);
    if (dot == DOT_ENC && enc_prec == WD_HALF_I16) return (void)WD_SPLIT(DOT_ENC, SI16);
    if (dot == DOT_ENC) return (void)WD_SPLIT(DOT_ENC, SF16);
  }
  WD_SPLIT(DOT_NONE, S);
#undef WD_SPLIT
}

template <class S, int RECON, int BASIS, int HPW>
static void launch_split_recon(const wd_gauge* gg, const DslashArgs& d, const LaunchCfg& c, hipStream_t s) {
  DslashGeom g = make_split_geom(gg->geom, d.rhs_map ? d.n_map : d.out.nrhs, c);
  g.mapped = d.rhs_map ? 1 : 0;
  g.tgauge = gg->tgauge;
  const char* links = static_cast<const char*>(gg->link[S::prec]);
  const unsigned grid = grid_blocks(g);
  const FieldView fo = fview(d.out), fi = fview(d.in), fx = fview(d.xpay), fy = fview(d.y);
  const auto ar = static_cast<typename S::real>(d.a);
  const int dot = d.xpay ? d.dot : DOT_NONE;
  EncView ev{fview(d.enc_rh), fview(d.enc_xh), fview(d.enc_rt), d.enc_set_rt, FinArgs{-1}};
  if (d.finalized) {
    *d.finalized = dot != DOT_NONE && d.fin.stage >= 0 && (g.slab ? 8 : 1) * g.site_blocks <= kFusedRecords;
    if (*d.finalized) ev.fin = d.fin;
  }
  const int* sel = d.rhs_map ? d.rhs_map : d.active;
  if (d.dagger) {
    if (d.xpay) launch_split_dot<S, true, true, RECON, BASIS, HPW>(dot, grid, s, g, links, fo, fi, fx, fy, ar, d.out_parity, sel, d.wave_partials, ev, d.enc_prec);
    else launch_split_dot<S, true, false, RECON, BASIS, HPW>(dot, grid, s, g, links, fo, fi, fx, fy, ar, d.out_parity, sel, d.wave_partials, ev, d.enc_prec);
  } else {
    if (d.xpay) launch_split_dot<S, false, true, RECON, BASIS, HPW>(dot, grid, s, g, links, fo, fi, fx, fy, ar, d.out_parity, sel, d.wave_partials, ev, d.enc_prec);
    else launch_split_dot<S, false, false, RECON, BASIS, HPW>(dot, grid, s, g, links, fo, fi, fx, fy, ar, d.out_parity, sel, d.wave_partials, ev, d.enc_prec);
  }
}

template <class S, int BASIS>
static void launch_split(const wd_gauge* gg, const DslashArgs& d, const LaunchCfg& c, hipStream_t s) {
  if constexpr (S::prec == WD_FP64) {
    if ((int64_t)gg->geom.Vh * (d.rhs_map ? d.n_map : d.out.nrhs) > 65536) {
      if (gg->recon == 8) launch_split_recon<S, 8, BASIS, 2>(gg, d, c, s);
      else launch_split_recon<S, 12, BASIS, 2>(gg, d, c, s);
      return;
    }
  }
  if (gg->recon == 8) launch_split_recon<S, 8, BASIS, 1>(gg, d, c, s);
  else launch_split_recon<S, 12, BASIS, 1>(gg, d, c, s);
}

}  // namespace wd
