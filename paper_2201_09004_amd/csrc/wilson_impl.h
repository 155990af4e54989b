// Wilson-type hopping stencil (sec. 2.1, eq. 2; sec. 2.3 for H_W) with fused
// epilogues, for FP64 / FP32 / FP16 storage and full or reconstructed links.
//
// For output parity p the kernel computes, per site x and column,
//   hop(x) = sum_mu [(1 - g_mu) U_mu(x) psi(x+mu) + (1 + g_mu) U_mu^dag(x-mu) psi(x-mu)]
// reading psi on parity 1-p (the dagger swaps the two projectors), then one of
//   EPI_HOP         out = k hop
//   EPI_XPAY        out = a x + k hop                 (Wilson D)
//   EPI_XPAY_NORM   the same and |out|^2              (CG on D^dag D: <p, D^dag D p> = |D p|^2)
//   EPI_XPAY_G5     out = g5 (a x + k hop)            (H_W = g5 D_W(-rho), sec. 2.3)
//   EPI_CLOVINV     out = A^{-1} (k hop)              (first half of the Schur operator)
//   EPI_CLOVINV_XPAY out = A^{-1} (x + k hop)         (even-odd source, odd-site reconstruction)
//   EPI_XMY_CLOVINV out = x - A^{-1} (k hop)          (second half)
//   EPI_CLOVINV_ACC out = v + A^{-1} (x + k hop)      (the same, onto the multigrid correction)
//   EPI_RESID       out = v - (A x + k hop)           (residual of the full twisted-clover D)
//   EPI_SITE        out = A x + k hop,  A = H + i mu g5 (full twisted-clover D)
//   EPI_CHEB        out = s1 g5 (a x + k hop) + ck v + s2 b1 - b2   (one Clenshaw step)
// where x, v, b1, b2 are fields of the output parity.  The time-boundary
// sign is applied here from the coordinates, so links stay exactly SU(3)
// for the 12-real reconstruction.
//
// Register blocking: one thread owns one site and NR consecutive columns, so
// each link and each site matrix is loaded once and used NR times.  Every
// column is computed with the same arithmetic in the same order whatever NR
// is, so all NR variants give bitwise-identical results.
//
// Spin projection in the chiral basis g_mu = [[0, P_mu], [P_mu^dag, 0]],
// P_k = -i sigma_k, P_4 = 1: (1 + s g_mu) psi = (h, s P_mu^dag h) with
// h = psi_up + s P_mu psi_low, so only two colour vectors meet the link.
#pragma once

#include "lq_common.h"
#include "lq_kernels.h"

namespace lq {

template <int MU, int S, typename R>
__device__ __forceinline__ void project(const cx<R>* p, cx<R>* h) {
  const R s = (R)S;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    cx<R> p0 = p[a], p1 = p[3 + a], p2 = p[6 + a], p3 = p[9 + a];
    if constexpr (MU == 0) {
      h[a] = p0 + s * times_mi(p3);
      h[3 + a] = p1 + s * times_mi(p2);
    } else if constexpr (MU == 1) {
      h[a] = p0 - s * p3;
      h[3 + a] = p1 + s * p2;
    } else if constexpr (MU == 2) {
      h[a] = p0 + s * times_mi(p2);
      h[3 + a] = p1 + s * times_i(p3);
    } else {
      h[a] = p0 + s * p2;
      h[3 + a] = p1 + s * p3;
    }
  }
}

template <int MU, int S, typename R>
__device__ __forceinline__ void recon_add(cx<R>* o, const cx<R>* h) {
  const R s = (R)S;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    cx<R> h0 = h[a], h1 = h[3 + a];
    o[a] = o[a] + h0;
    o[3 + a] = o[3 + a] + h1;
    if constexpr (MU == 0) {
      o[6 + a] = o[6 + a] + s * times_i(h1);
      o[9 + a] = o[9 + a] + s * times_i(h0);
    } else if constexpr (MU == 1) {
      o[6 + a] = o[6 + a] + s * h1;
      o[9 + a] = o[9 + a] - s * h0;
    } else if constexpr (MU == 2) {
      o[6 + a] = o[6 + a] + s * times_i(h0);
      o[9 + a] = o[9 + a] + s * times_mi(h1);
    } else {
      o[6 + a] = o[6 + a] + s * h0;
      o[9 + a] = o[9 + a] + s * h1;
    }
  }
}

// the forward (x + mu) hop of one direction for NR columns starting at col0
template <int P, int NE, bool DAG, int MU, int NR, typename R>
__device__ __forceinline__ void hop_fwd(const WilsonArgs& A, const int c[4], int par, int cb, int col0, int nv,
                                        cx<R> (*acc)[12]) {
  const Geom& g = A.g;
  const int pin = par ^ 1;
  cx<R> U[9];
  const int nb = neighbour<P, MU, 1>(c, cb, g);
  load_link<P, NE>(A.links, g.Vh, par, MU, cb, U);
  const bool flip = (MU == 3 && g.ap && c[3] == g.L[3] - 1);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (r < nv) {
      cx<R> psi[12], h[6], uh[6];
      IO<P, 12>::load(A.in, blk_index(A.in, col0 + r, pin), nb, psi);
      project<MU, DAG ? 1 : -1>(psi, h);
      if (flip) {
#pragma unroll
        for (int i = 0; i < 6; ++i) h[i] = -h[i];
      }
      su3_mv(U, h, uh);
      su3_mv(U, h + 3, uh + 3);
      recon_add<MU, DAG ? 1 : -1>(acc[r], uh);
    }
  }
}

// the backward (x - mu) hop
template <int P, int NE, bool DAG, int MU, int NR, typename R>
__device__ __forceinline__ void hop_bwd(const WilsonArgs& A, const int c[4], int par, int cb, int col0, int nv,
                                        cx<R> (*acc)[12]) {
  const Geom& g = A.g;
  const int pin = par ^ 1;
  cx<R> U[9];
  const int nb = neighbour<P, MU, -1>(c, cb, g);
  load_link<P, NE>(A.links, g.Vh, pin, MU, nb, U);
  const bool flip = (MU == 3 && g.ap && c[3] == 0);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (r < nv) {
      cx<R> psi[12], h[6], uh[6];
      IO<P, 12>::load(A.in, blk_index(A.in, col0 + r, pin), nb, psi);
      project<MU, DAG ? -1 : 1>(psi, h);
      if (flip) {
#pragma unroll
        for (int i = 0; i < 6; ++i) h[i] = -h[i];
      }
      su3_mv_dag(U, h, uh);
      su3_mv_dag(U, h + 3, uh + 3);
      recon_add<MU, DAG ? -1 : 1>(acc[r], uh);
    }
  }
}

// ------------------------------------------------------------ FP16 hops
// Vector instructions took most of a full-volume launch (3356 per site and two
// columns, 90% of its time at one per 4 cycles and wave), so the hops read halves
// where they are used.  v_fma_mix_f32 takes an FP16 operand as an exact FP32 one:
// the projection is one such instruction per real number, fma(a, 1, +-b) on
// the halves of two spins, the links are multiplied as halves, and the site's
// norm (with k_hop and the time-boundary sign) scales the transported vector
// in the FMA that adds it up.  All sums and products are FP32, and fewer of
// them round than with every half scaled by its norm first (the sign function of
// order 200 is as far from FP64 as before, 8.175e-4 at 24^3x64, its FP16 state
// being what rounds).  That leaves 2585, and traffic bounds the launch now: 2.5 GB
// across the L2 boundary for 1.36 GB of operands (the Clenshaw step 4.0 for 2.46)
// at 5.1 - 5.5 TB/s.  12 columns at 24^3x64: g5 (a x + k hop) 592 -> 486 us, the
// Clenshaw step 773 -> 722 us.
struct Half2 {
  _Float16 re, im;
};
__device__ __forceinline__ float re32(Half2 z) { return (float)z.re; }
__device__ __forceinline__ float im32(Half2 z) { return (float)z.im; }
__device__ __forceinline__ float re32(cx<float> z) { return z.re; }
__device__ __forceinline__ float im32(cx<float> z) { return z.im; }
__device__ __forceinline__ Half2 half2_of(unsigned w) {
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  const h2 h = __builtin_bit_cast(h2, w);
  return {h.x, h.y};
}
struct Spin16 {
  Half2 p[12];
  float n;
};
// Column col's spinor at site cb of parity par.  The column's part of the
// address is a scalar and the parity's a select, so that a lane multiplies for
// neither (integer multiplications issue at a quarter of the rate).
__device__ __forceinline__ Spin16 load_spin16(const FieldRef& f, int col, int par, int cb) {
  const int64_t pv = f.npar == 2 && par ? f.Vh : 0;  // sites before this parity's in the column
  const uint4* p = (const uint4*)f.data + tix((int64_t)col * f.npar, 0, 3, 0, f.Vh) + (pv * 3 + tix(0, 0, 3, cb, f.Vh));
  Spin16 s;
  s.n = f.norm[(int64_t)col * f.npar * f.Vh + (pv + cb)];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint4 d = p[tix(0, k, 3, 0, f.Vh)];
    s.p[4 * k] = half2_of(d.x);
    s.p[4 * k + 1] = half2_of(d.y);
    s.p[4 * k + 2] = half2_of(d.z);
    s.p[4 * k + 3] = half2_of(d.w);
  }
  return s;
}
// (1 + S g_mu) psi, upper spins; one = 1 behind an asm barrier, so that the sums stay fma_mix
template <int MU, int S>
__device__ __forceinline__ void project16(const Half2* p, float one, cx<float>* h) {
  constexpr float s = (float)S;
#define LQ_MIX(A, SG, B) __builtin_fmaf((float)(A), one, (SG) * (float)(B))
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const Half2 p0 = p[a], p1 = p[3 + a], p2 = p[6 + a], p3 = p[9 + a];
    if constexpr (MU == 0) {
      h[a] = {LQ_MIX(p0.re, s, p3.im), LQ_MIX(p0.im, -s, p3.re)};
      h[3 + a] = {LQ_MIX(p1.re, s, p2.im), LQ_MIX(p1.im, -s, p2.re)};
    } else if constexpr (MU == 1) {
      h[a] = {LQ_MIX(p0.re, -s, p3.re), LQ_MIX(p0.im, -s, p3.im)};
      h[3 + a] = {LQ_MIX(p1.re, s, p2.re), LQ_MIX(p1.im, s, p2.im)};
    } else if constexpr (MU == 2) {
      h[a] = {LQ_MIX(p0.re, s, p2.im), LQ_MIX(p0.im, -s, p2.re)};
      h[3 + a] = {LQ_MIX(p1.re, -s, p3.im), LQ_MIX(p1.im, s, p3.re)};
    } else {
      h[a] = {LQ_MIX(p0.re, s, p2.re), LQ_MIX(p0.im, s, p2.im)};
      h[3 + a] = {LQ_MIX(p1.re, s, p3.re), LQ_MIX(p1.im, s, p3.im)};
    }
  }
#undef LQ_MIX
}
// o += n (1 + S g_mu) h
template <int MU, int S>
__device__ __forceinline__ void recon16(cx<float>* o, float n, const cx<float>* h) {
  const float m = S * n;
  auto add = [](cx<float>& a, float f, cx<float> z) {  // a += f z
    a.re = __builtin_fmaf(f, z.re, a.re);
    a.im = __builtin_fmaf(f, z.im, a.im);
  };
  auto add_i = [](cx<float>& a, float f, cx<float> z) {  // a += i f z
    a.re = __builtin_fmaf(-f, z.im, a.re);
    a.im = __builtin_fmaf(f, z.re, a.im);
  };
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cx<float> h0 = h[a], h1 = h[3 + a];
    add(o[a], n, h0);
    add(o[3 + a], n, h1);
    if constexpr (MU == 0) {
      add_i(o[6 + a], m, h1);
      add_i(o[9 + a], m, h0);
    } else if constexpr (MU == 1) {
      add(o[6 + a], m, h1);
      add(o[9 + a], -m, h0);
    } else if constexpr (MU == 2) {
      add_i(o[6 + a], m, h0);
      add_i(o[9 + a], -m, h1);
    } else {
      add(o[6 + a], m, h0);
      add(o[9 + a], m, h1);
    }
  }
}
// y = U x (ADJ: U^dag x) for the two colour vectors of x
template <bool ADJ, typename E>
__device__ __forceinline__ void link16(const E* U, const cx<float>* x, cx<float>* y) {
#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cx<float> s = {0.f, 0.f};
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const E u = ADJ ? U[3 * b + a] : U[3 * a + b];
        const cx<float> z = x[3 * v + b];
        const float ur = re32(u), ui = ADJ ? -im32(u) : im32(u);
        s.re = __builtin_fmaf(ur, z.re, s.re);
        s.re = __builtin_fmaf(-ui, z.im, s.re);
        s.im = __builtin_fmaf(ur, z.im, s.im);
        s.im = __builtin_fmaf(ui, z.re, s.im);
      }
      y[3 * v + a] = s;
    }
}
// one hop (FWD: x + mu) of NR columns; k = k_hop times what the epilogue scales the sum by
template <int NE, bool FWD, int S, int MU, int NR>
__device__ __forceinline__ void hop16(const WilsonArgs& A, const int c[4], int par, int cb, int col0, int nv, float k,
                                      float one, cx<float> (*acc)[12]) {
  const Geom& g = A.g;
  const int pin = par ^ 1, nb = nb_cb<MU, FWD ? 1 : -1>(c, cb, g);
  const int lpar = FWD ? par : pin, lcb = FWD ? cb : nb;
  const bool flip = MU == 3 && g.ap && c[3] == (FWD ? g.L[3] - 1 : 0);
  const float kk = flip ? -k : k;
  auto columns = [&](const auto* U) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (r < nv) {
        const Spin16 x = load_spin16(A.in, col0 + r, pin, nb);
        cx<float> h[6], uh[6];
        project16<MU, S>(x.p, one, h);
        link16<!FWD>(U, h, uh);
        recon16<MU, S>(acc[r], kk * x.n, uh);
      }
    }
  };
  if constexpr (NE == 9) {
    const unsigned* p = (const unsigned*)A.links + tix(MU, 0, 9, 0, g.Vh) +
                        ((lpar ? 4 * (int64_t)g.Vh : 0) * 9 + tix(0, 0, 9, lcb, g.Vh));
    Half2 U[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) U[e] = half2_of(p[tix(0, e, 9, 0, g.Vh)]);
    columns(U);
  } else {
    cx<float> U[9];
    load_link<16, NE>(A.links, g.Vh, lpar, MU, lcb, U);
    columns(U);
  }
}
// acc = k hop(x), in the hop order of wilson_kernel
template <int NE, bool DAG, int NR>
__device__ __forceinline__ void hops16(const WilsonArgs& A, const int c[4], int par, int cb, int col0, int nv, float k,
                                       cx<float> (*acc)[12]) {
  constexpr int B = DAG ? -1 : 1;
  float one = 1.0f;
  asm volatile("" : "+s"(one));
  hop16<NE, false, B, 3, NR>(A, c, par, cb, col0, nv, k, one, acc);
  hop16<NE, false, B, 2, NR>(A, c, par, cb, col0, nv, k, one, acc);
  hop16<NE, false, B, 1, NR>(A, c, par, cb, col0, nv, k, one, acc);
  hop16<NE, false, B, 0, NR>(A, c, par, cb, col0, nv, k, one, acc);
  hop16<NE, true, -B, 0, NR>(A, c, par, cb, col0, nv, k, one, acc);
  hop16<NE, true, -B, 1, NR>(A, c, par, cb, col0, nv, k, one, acc);
  hop16<NE, true, -B, 2, NR>(A, c, par, cb, col0, nv, k, one, acc);
  hop16<NE, true, -B, 3, NR>(A, c, par, cb, col0, nv, k, one, acc);
}
// o += f psi of the output site (halves read in the FMA)
__device__ __forceinline__ void axpy16(const FieldRef& x, int col, int par, int cb, float f, cx<float>* o) {
  const Spin16 s = load_spin16(x, col, par, cb);
  const float m = f * s.n;
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    o[i].re = __builtin_fmaf(m, (float)s.p[i].re, o[i].re);
    o[i].im = __builtin_fmaf(m, (float)s.p[i].im, o[i].im);
  }
}

// 6x6 complex matrix [36] (row-major) times the chiral halves of NR columns, each
// matrix entry loaded once; in place on v[r][off..off+5]
template <int P, int NR, typename R>
__device__ __forceinline__ void apply_full6_nr(const void* base, int Vh, int par, int chir, int cb, int nv,
                                               cx<R> (*v)[12], int off) {
  using T2 = typename LinkT<P>::T2;
  const T2* p = (const T2*)base;
  const int g = par * 2 + chir;
  cx<R> y[NR][6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
#pragma unroll
    for (int r = 0; r < NR; ++r) y[r][i] = {0, 0};
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      T2 d = ldx<true>(p + tix(g, i * 6 + j, 36, cb, Vh));
      const cx<R> m = {(R)d.x, (R)d.y};
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (r < nv) fma(y[r][i], m, v[r][off + j]);
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int i = 0; i < 6; ++i) v[r][off + i] = y[r][i];
}

// Hermitian 6x6 packed as 3 T2 of diagonal pairs + 15 lower entries (i>j, row order)
template <int P, typename R>
__device__ __forceinline__ void apply_herm6(const void* base, int Vh, int par, int chir, int cb, const cx<R>* v,
                                            cx<R>* y) {
  using T2 = typename LinkT<P>::T2;
  const T2* p = (const T2*)base;
  const int g = par * 2 + chir;
  R d[6];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    T2 e = ldx<true>(p + tix(g, k, 18, cb, Vh));
    d[2 * k] = (R)e.x;
    d[2 * k + 1] = (R)e.y;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) y[i] = d[i] * v[i];
  int k = 3;
#pragma unroll
  for (int i = 1; i < 6; ++i) {
#pragma unroll
    for (int j = 0; j < i; ++j) {
      T2 e = ldx<true>(p + tix(g, k, 18, cb, Vh));
      ++k;
      cx<R> l = {(R)e.x, (R)e.y};
      fma(y[i], l, v[j]);
      fmac(y[j], l, v[i]);
    }
  }
}

// Minimum waves per SIMD asked of the compiler for the FP64 / FP32 variants (the
// register-blocked ones use up to 256 VGPRs; 1 leaves the register budget
// at 256 and occupancy at 2 waves).
#ifndef LQ_MINW64
#define LQ_MINW64 1
#endif
#ifndef LQ_MINW32
#define LQ_MINW32 1
#endif
template <int P, int NE, bool DAG, int EPI, int NR>
__global__ void __attribute__((amdgpu_flat_work_group_size(1, kStencilMaxThreads),
                               amdgpu_waves_per_eu(P == 64 ? LQ_MINW64 : P == 32 ? LQ_MINW32 : 1)))
wilson_kernel(WilsonArgs A) {
  using R = typename RealOf<P>::T;
  constexpr bool XMY = EPI == EPI_XMY_CLOVINV || EPI == EPI_XMY_RTS;
  constexpr bool RED = EPI == EPI_XMY_RTS || EPI == EPI_XPAY_NORM;
  if (A.ncol <= 0) return;
  const int ngrp = (A.ncol + NR - 1) / NR;
  int par, cb, grp, c[4], tile = 0;
  const int status = stencil_site(A.g, A.par_out, A.slab, ngrp, A.sh, par, cb, grp, c, &tile);
  // lanes past the end of the last tile stay only to join the wave reductions
  if (status == 0 || (!RED && status != 1)) return;
  const bool live = status == 1;
  const int col0 = grp * NR;
  const int nv = min(NR, A.ncol - col0);  // <= 0 for waves without columns

  cx<R> acc[NR][12];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int i = 0; i < 12; ++i) acc[r][i] = {0, 0};
  // Hop order: the backward hops from t down to x, then the forward hops from
  // x up to t.  A spinor that one wave reads as its +mu neighbour is read as
  // the -mu neighbour by a wave started later (its tile lies further along
  // the traversal); reading -mu early and +mu late brings the two reads
  // closer in time, most for t, whose neighbours are furthest apart, so more
  // of the second reads hit L2 (3% on the 12-column FP32 Schur stencils
  // against forward-backward per direction).
  if constexpr (P == 16) {
    hops16<NE, DAG, NR>(A, c, par, cb, col0, nv, (float)(EPI == EPI_CHEB ? A.s1 * A.k_hop : A.k_hop), acc);
  } else {
    hop_bwd<P, NE, DAG, 3, NR>(A, c, par, cb, col0, nv, acc);
    hop_bwd<P, NE, DAG, 2, NR>(A, c, par, cb, col0, nv, acc);
    hop_bwd<P, NE, DAG, 1, NR>(A, c, par, cb, col0, nv, acc);
    hop_bwd<P, NE, DAG, 0, NR>(A, c, par, cb, col0, nv, acc);
    hop_fwd<P, NE, DAG, 0, NR>(A, c, par, cb, col0, nv, acc);
    hop_fwd<P, NE, DAG, 1, NR>(A, c, par, cb, col0, nv, acc);
    hop_fwd<P, NE, DAG, 2, NR>(A, c, par, cb, col0, nv, acc);
    hop_fwd<P, NE, DAG, 3, NR>(A, c, par, cb, col0, nv, acc);

    const R k = (R)A.k_hop;
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int i = 0; i < 12; ++i) acc[r][i] = k * acc[r][i];
  }

  if constexpr (EPI == EPI_CLOVINV_XPAY || EPI == EPI_CLOVINV_ACC) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (r >= nv) continue;
      cx<R> x[12];
      IO<P, 12>::template load<true>(A.x, blk_index(A.x, col0 + r, par), cb, x);
#pragma unroll
      for (int i = 0; i < 12; ++i) acc[r][i] = acc[r][i] + x[i];
    }
  }
  if constexpr (EPI == EPI_CLOVINV || XMY || EPI == EPI_CLOVINV_XPAY || EPI == EPI_CLOVINV_ACC) {
    apply_full6_nr<P, NR>(A.clov_inv, A.g.Vh, par, 0, cb, nv, acc, 0);
    apply_full6_nr<P, NR>(A.clov_inv, A.g.Vh, par, 1, cb, nv, acc, 6);
  }
  double red[NR][3];
#pragma unroll
  for (int r = 0; r < NR; ++r) red[r][0] = red[r][1] = red[r][2] = 0.0;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (r >= nv) continue;
    const int col = col0 + r;
    cx<R> out[12];
    if constexpr (EPI == EPI_HOP || EPI == EPI_CLOVINV || EPI == EPI_CLOVINV_XPAY) {
#pragma unroll
      for (int i = 0; i < 12; ++i) out[i] = acc[r][i];
    } else if constexpr (EPI == EPI_CLOVINV_ACC) {
      cx<R> v[12];
      IO<P, 12>::template load<true>(A.v, blk_index(A.v, col, par), cb, v);
#pragma unroll
      for (int i = 0; i < 12; ++i) out[i] = v[i] + acc[r][i];
    } else if constexpr (XMY) {
      cx<R> x[12];
      IO<P, 12>::template load<true>(A.x, blk_index(A.x, col, par), cb, x);
#pragma unroll
      for (int i = 0; i < 12; ++i) out[i] = x[i] - acc[r][i];
      if (live) {
        if constexpr (RED) {
#pragma unroll
          for (int i = 0; i < 12; ++i) {
            red[r][0] += (double)out[i].re * (double)x[i].re + (double)out[i].im * (double)x[i].im;
            red[r][1] += (double)out[i].re * (double)x[i].im - (double)out[i].im * (double)x[i].re;
            red[r][2] += (double)out[i].re * (double)out[i].re + (double)out[i].im * (double)out[i].im;
          }
        }
      }
    } else if constexpr (EPI == EPI_XPAY || EPI == EPI_XPAY_NORM || EPI == EPI_XPAY_G5 || EPI == EPI_CHEB) {
      const R a = A.acol ? (R)A.acol[col] : (R)A.a;
      if constexpr (P == 16) {
#pragma unroll
        for (int i = 0; i < 12; ++i) out[i] = acc[r][i];
        axpy16(A.x, col, par, cb, EPI == EPI_CHEB ? (float)A.s1 * a : a, out);
      } else {
        cx<R> x[12];
        IO<P, 12>::template load<true>(A.x, blk_index(A.x, col, par), cb, x);
#pragma unroll
        for (int i = 0; i < 12; ++i) out[i] = a * x[i] + acc[r][i];
      }
      if constexpr (EPI == EPI_XPAY_NORM) {
        if (live) {
#pragma unroll
          for (int i = 0; i < 12; ++i)
            red[r][0] += (double)out[i].re * (double)out[i].re + (double)out[i].im * (double)out[i].im;
        }
      }
      if constexpr (EPI == EPI_XPAY_G5 || EPI == EPI_CHEB) {
#pragma unroll
        for (int i = 6; i < 12; ++i) out[i] = -out[i];
      }
      if constexpr (EPI == EPI_CHEB && P == 16) {
        axpy16(A.v, col, par, cb, (float)A.ck, out);
        axpy16(A.b1, col, par, cb, (float)A.s2, out);
        axpy16(A.b2, col, par, cb, -1.0f, out);
      } else if constexpr (EPI == EPI_CHEB) {
        cx<R> v[12];
        const R s1 = (R)A.s1, ck = (R)A.ck, s2 = (R)A.s2;
        IO<P, 12>::template load<true>(A.v, blk_index(A.v, col, par), cb, v);
#pragma unroll
        for (int i = 0; i < 12; ++i) out[i] = s1 * out[i] + ck * v[i];
        IO<P, 12>::template load<true>(A.b1, blk_index(A.b1, col, par), cb, v);
#pragma unroll
        for (int i = 0; i < 12; ++i) out[i] = out[i] + s2 * v[i];
        IO<P, 12>::template load<true>(A.b2, blk_index(A.b2, col, par), cb, v);
#pragma unroll
        for (int i = 0; i < 12; ++i) out[i] = out[i] - v[i];
      }
    } else if constexpr (EPI == EPI_SITE || EPI == EPI_RESID) {
      cx<R> x[12];
      IO<P, 12>::template load<true>(A.x, blk_index(A.x, col, par), cb, x);
      apply_herm6<P>(A.clov, A.g.Vh, par, 0, cb, x, out);
      apply_herm6<P>(A.clov, A.g.Vh, par, 1, cb, x + 6, out + 6);
      const R mu = (R)A.mu_tw;
#pragma unroll
      for (int i = 0; i < 6; ++i) out[i] = out[i] + mu * times_i(x[i]) + acc[r][i];
#pragma unroll
      for (int i = 6; i < 12; ++i) out[i] = out[i] - mu * times_i(x[i]) + acc[r][i];
      if constexpr (EPI == EPI_RESID) {
        IO<P, 12>::template load<true>(A.v, blk_index(A.v, col, par), cb, x);
#pragma unroll
        for (int i = 0; i < 12; ++i) out[i] = x[i] - out[i];
      }
    }
    if (live) IO<P, 12>::template store<true>(A.out, blk_index(A.out, col, par), cb, out);
  }
  if constexpr (RED) {
    // wave butterfly (fixed order) and one partial per (column, 64-site tile)
    const int nsite = A.par_out == 2 ? 2 * A.g.Vh : A.g.Vh;
    const int ntile = (nsite + 63) >> 6;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (r >= nv) continue;
#pragma unroll
      for (int k = 0; k < 3; ++k)
        for (int o = 32; o > 0; o >>= 1) red[r][k] += __shfl_xor(red[r][k], o);
      if ((threadIdx.x & 63) == 0) {
        double* p = A.red + ((int64_t)(col0 + r) * ntile + tile) * 4;
        p[0] = red[r][0];
        p[1] = red[r][1];
        p[2] = red[r][2];
        p[3] = 0.0;
      }
    }
  }
}

// ------------------------------------------------------------ small launches
// The same operators for launches of few waves, where the chain of one
// thread's eight hops is what takes the time (4096 sites are 64 waves on 1024
// SIMDs): a workgroup of eight waves takes 64 sites and one column, each wave
// one hop, the two transported colour vectors of every hop meet in LDS, and
// four waves, one spin each (two, one chirality each, where the site matrix
// couples the spins), sum them in the hop order of wilson_kernel and finish.  The arithmetic of every element is the same in the same order, so
// the results are bitwise those of wilson_kernel and the tuner may choose.
// 8^4, one column, FP64: twisted-clover D 11.7 -> 7.0 us, Wilson D with |out|^2
// 7.9 -> 5.8 us, D^dag 7.0 -> 5.1 us.
template <int P> __device__ __forceinline__ cx<typename RealOf<P>::T> load_comp(const FieldRef& f, int64_t blk, int cb, int c) {
  static_assert(P != 16, "FP16 sites are whole");
  if constexpr (P == 64) {
    const double2 v = ((const double2*)f.data)[tix(blk, c, 12, cb, f.Vh)];
    return {v.x, v.y};
  } else {
    const float2 v = ((const float2*)f.data)[2 * tix(blk, c >> 1, 6, cb, f.Vh) + (c & 1)];
    return {v.x, v.y};
  }
}
template <int P> __device__ __forceinline__ void store_comp(const FieldRef& f, int64_t blk, int cb, int c, cx<typename RealOf<P>::T> v) {
  if constexpr (P == 64) ((double2*)f.data)[tix(blk, c, 12, cb, f.Vh)] = make_double2(v.re, v.im);
  else ((float2*)f.data)[2 * tix(blk, c >> 1, 6, cb, f.Vh) + (c & 1)] = make_float2(v.re, v.im);
}

// U h or U^dag h of the hop by S along MU
template <int P, int NE, bool DAG, int MU, int S, typename R>
__device__ __forceinline__ void split_hop(const WilsonArgs& A, const int c[4], int par, int cb, int col, cx<R>* uh) {
  const Geom& g = A.g;
  const int pin = par ^ 1;
  cx<R> U[9], psi[12], h[6];
  const int nb = nb_cb<MU, S>(c, cb, g);
  load_link<P, NE>(A.links, g.Vh, S > 0 ? par : pin, MU, S > 0 ? cb : nb, U);
  IO<P, 12>::load(A.in, blk_index(A.in, col, pin), nb, psi);
  project<MU, (S > 0) == DAG ? 1 : -1>(psi, h);
  if (MU == 3 && g.ap && c[3] == (S > 0 ? g.L[3] - 1 : 0)) {
#pragma unroll
    for (int i = 0; i < 6; ++i) h[i] = -h[i];
  }
  if constexpr (S > 0) {
    su3_mv(U, h, uh);
    su3_mv(U, h + 3, uh + 3);
  } else {
    su3_mv_dag(U, h, uh);
    su3_mv_dag(U, h + 3, uh + 3);
  }
}

// spin W's part of recon_add for the hop along MU with projector sign SP
template <int MU, int SP, int W, typename R>
__device__ __forceinline__ void split_add(cx<R>* o, const cx<R> (*uh)[64], int lane) {
  const R s = (R)SP;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if constexpr (W < 2) {
      o[a] = o[a] + uh[3 * W + a][lane];
    } else if constexpr (MU == 0) {
      o[a] = o[a] + s * times_i(uh[W == 2 ? 3 + a : a][lane]);
    } else if constexpr (MU == 1) {
      if constexpr (W == 2) o[a] = o[a] + s * uh[3 + a][lane];
      else o[a] = o[a] - s * uh[a][lane];
    } else if constexpr (MU == 2) {
      if constexpr (W == 2) o[a] = o[a] + s * times_i(uh[a][lane]);
      else o[a] = o[a] + s * times_mi(uh[3 + a][lane]);
    } else {
      o[a] = o[a] + s * uh[W == 2 ? a : 3 + a][lane];
    }
  }
}

// the scaled hop sum of spin W
template <bool DAG, int W, typename R>
__device__ __forceinline__ void split_sum(const WilsonArgs& A, int lane, const cx<R> (*sm)[6][64], cx<R>* acc) {
  constexpr int SB = DAG ? -1 : 1;  // projector sign of the backward hops
#pragma unroll
  for (int a = 0; a < 3; ++a) acc[a] = {0, 0};
  split_add<3, SB, W>(acc, sm[0], lane);
  split_add<2, SB, W>(acc, sm[1], lane);
  split_add<1, SB, W>(acc, sm[2], lane);
  split_add<0, SB, W>(acc, sm[3], lane);
  split_add<0, -SB, W>(acc, sm[4], lane);
  split_add<1, -SB, W>(acc, sm[5], lane);
  split_add<2, -SB, W>(acc, sm[6], lane);
  split_add<3, -SB, W>(acc, sm[7], lane);
  const R k = (R)A.k_hop;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    acc[a] = k * acc[a];
    // rounded here, as in wilson_kernel: the sums that follow fuse their other product
    asm volatile("" : "+v"(acc[a].re), "+v"(acc[a].im));
  }
}

// one spin of every epilogue without site matrices
template <int P, bool DAG, int EPI, int W, typename R>
__device__ __forceinline__ void split_finish(const WilsonArgs& A, int par, int cb, int col, int lane, bool live,
                                             const cx<R> (*sm)[6][64], cx<R>* out) {
  cx<R> acc[3];
  split_sum<DAG, W>(A, lane, sm, acc);
  if constexpr (EPI == EPI_HOP) {
#pragma unroll
    for (int a = 0; a < 3; ++a) out[a] = acc[a];
  } else {
    const R s = A.acol ? (R)A.acol[col] : (R)A.a;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const cx<R> x = load_comp<P>(A.x, blk_index(A.x, col, par), cb, 3 * W + a);
      out[a] = s * x + acc[a];
      if constexpr (EPI == EPI_XPAY_G5 && W >= 2) out[a] = -out[a];
    }
  }
  if (live) {
#pragma unroll
    for (int a = 0; a < 3; ++a) store_comp<P>(A.out, blk_index(A.out, col, par), cb, 3 * W + a, out[a]);
  }
}

// one chirality of EPI_SITE
template <int P, bool DAG, int CH, typename R>
__device__ __forceinline__ void split_site(const WilsonArgs& A, int par, int cb, int col, int lane, bool live,
                                           const cx<R> (*sm)[6][64]) {
  cx<R> acc[6], x[6], out[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) x[i] = load_comp<P>(A.x, blk_index(A.x, col, par), cb, 6 * CH + i);
  split_sum<DAG, 2 * CH>(A, lane, sm, acc);
  split_sum<DAG, 2 * CH + 1>(A, lane, sm, acc + 3);
  apply_herm6<P>(A.clov, A.g.Vh, par, CH, cb, x, out);
  const R mu = (R)A.mu_tw;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    if constexpr (CH == 0) out[i] = out[i] + mu * times_i(x[i]) + acc[i];
    else out[i] = out[i] - mu * times_i(x[i]) + acc[i];
    if (live) store_comp<P>(A.out, blk_index(A.out, col, par), cb, 6 * CH + i, out[i]);
  }
}

template <int P, int NE, bool DAG, int EPI>
__global__ void __launch_bounds__(512) wilson_split_kernel(WilsonArgs A) {
  using R = typename RealOf<P>::T;
  __shared__ cx<R> sm[8][6][64];
  const Geom& g = A.g;
  const int nsite = A.par_out == 2 ? 2 * g.Vh : g.Vh;
  const int tile = blockIdx.x, col = blockIdx.y, lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int j = tile * 64 + lane;
  const bool live = j < nsite;
  if (!live) j = nsite - 1;
  const int par = A.par_out == 2 ? (j >= g.Vh ? 1 : 0) : A.par_out;
  const int cb = A.par_out == 2 ? j - par * g.Vh : j;
  int c[4];
  cb_coords(cb, par, g, c);
  cx<R> uh[6];
  switch (w) {
    case 0: split_hop<P, NE, DAG, 3, -1>(A, c, par, cb, col, uh); break;
    case 1: split_hop<P, NE, DAG, 2, -1>(A, c, par, cb, col, uh); break;
    case 2: split_hop<P, NE, DAG, 1, -1>(A, c, par, cb, col, uh); break;
    case 3: split_hop<P, NE, DAG, 0, -1>(A, c, par, cb, col, uh); break;
    case 4: split_hop<P, NE, DAG, 0, 1>(A, c, par, cb, col, uh); break;
    case 5: split_hop<P, NE, DAG, 1, 1>(A, c, par, cb, col, uh); break;
    case 6: split_hop<P, NE, DAG, 2, 1>(A, c, par, cb, col, uh); break;
    default: split_hop<P, NE, DAG, 3, 1>(A, c, par, cb, col, uh); break;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) sm[w][i][lane] = uh[i];
  __syncthreads();
  if constexpr (EPI == EPI_SITE) {
    if (w == 0) split_site<P, DAG, 0>(A, par, cb, col, lane, live, sm);
    else if (w == 1) split_site<P, DAG, 1>(A, par, cb, col, lane, live, sm);
    return;
  }
  cx<R> out[3];
  switch (w) {
    case 0: split_finish<P, DAG, EPI, 0>(A, par, cb, col, lane, live, sm, out); break;
    case 1: split_finish<P, DAG, EPI, 1>(A, par, cb, col, lane, live, sm, out); break;
    case 2: split_finish<P, DAG, EPI, 2>(A, par, cb, col, lane, live, sm, out); break;
    case 3: split_finish<P, DAG, EPI, 3>(A, par, cb, col, lane, live, sm, out); break;
    default: break;
  }
  if constexpr (EPI == EPI_XPAY_NORM) {
    // |out|^2 of the tile, summed as in wilson_kernel: the site's twelve
    // components in order, then the butterfly over the sites
    __syncthreads();
    cx<R>(*o)[64] = &sm[0][0];
    if (w < 4)
#pragma unroll
      for (int a = 0; a < 3; ++a) o[3 * w + a][lane] = out[a];
    __syncthreads();
    if (w == 0) {
      double red = 0.0;
      if (live)
#pragma unroll
        for (int i = 0; i < 12; ++i) {
          const cx<R> v = o[i][lane];
          red += (double)v.re * (double)v.re + (double)v.im * (double)v.im;
        }
      for (int d = 32; d > 0; d >>= 1) red += __shfl_xor(red, d);
      if (lane == 0) {
        double* p = A.red + ((int64_t)col * ((nsite + 63) >> 6) + tile) * 4;
        p[0] = red;
        p[1] = p[2] = p[3] = 0.0;
      }
    }
  }
}

constexpr bool epi_split(int epi) {
  return epi == EPI_HOP || epi == EPI_XPAY || epi == EPI_XPAY_NORM || epi == EPI_XPAY_G5 || epi == EPI_SITE;
}
template <int P, int NE, bool DAG, int EPI>
inline int launch_split(const WilsonArgs& A, hipStream_t s) {
  const int nsite = A.par_out == 2 ? 2 * A.g.Vh : A.g.Vh;
  wilson_split_kernel<P, NE, DAG, EPI><<<dim3((nsite + 63) / 64, A.ncol), 512, 0, s>>>(A);
  return 0;
}

template <int P, int NE, bool DAG, int EPI, int NR>
inline void launch_one(const WilsonArgs& A, int bs, hipStream_t s) {
  (void)bs;
  const int nsite = A.par_out == 2 ? 2 * A.g.Vh : A.g.Vh;
  const StencilGrid G = stencil_grid(nsite, (A.ncol + NR - 1) / NR, A.tpb, A.xcd);
  WilsonArgs B = A;
  B.sh = G.sh;
  wilson_kernel<P, NE, DAG, EPI, NR><<<dim3(G.blocks), dim3(G.threads), 0, s>>>(B);
}

// epilogues with register-blocked variants (NR > 1)
constexpr bool epi_blocked(int epi) {
  return epi == EPI_CLOVINV || epi == EPI_XMY_CLOVINV || epi == EPI_XPAY || epi == EPI_XPAY_G5 || epi == EPI_CHEB ||
         epi == EPI_XMY_RTS || epi == EPI_SITE || epi == EPI_CLOVINV_XPAY || epi == EPI_XPAY_NORM ||
         epi == EPI_RESID || epi == EPI_CLOVINV_ACC;
}

template <int P, int NE, int EPI>
inline int launch_nr(const WilsonArgs& A, int nr, int bs, hipStream_t s) {
  if (nr == kSplitShape) {
    if constexpr (P != 16 && epi_split(EPI)) {
      if (!A.dag) return launch_split<P, NE, false, EPI>(A, s);
      if constexpr (EPI == EPI_XPAY || EPI == EPI_SITE) return launch_split<P, NE, true, EPI>(A, s);
    }
    nr = 1;
  }
  if (A.dag) {
    if constexpr (EPI == EPI_XPAY || EPI == EPI_SITE) {
      switch (nr) {
        case 2: launch_one<P, NE, true, EPI, 2>(A, bs, s); return 0;
        case 3: launch_one<P, NE, true, EPI, 3>(A, bs, s); return 0;
        case 4: launch_one<P, NE, true, EPI, 4>(A, bs, s); return 0;
        default: break;
      }
    }
    if (nr != 1) return -1;
    launch_one<P, NE, true, EPI, 1>(A, bs, s);
    return 0;
  }
  if constexpr (epi_blocked(EPI)) {
    switch (nr) {
      case 1: launch_one<P, NE, false, EPI, 1>(A, bs, s); return 0;
      case 2: launch_one<P, NE, false, EPI, 2>(A, bs, s); return 0;
      case 3: launch_one<P, NE, false, EPI, 3>(A, bs, s); return 0;
      case 4: launch_one<P, NE, false, EPI, 4>(A, bs, s); return 0;
      case 6:
        if constexpr (P != 64) {
          launch_one<P, NE, false, EPI, 6>(A, bs, s);
          return 0;
        }
        return -1;
      default: return -1;
    }
  }
  if (nr != 1) return -1;
  launch_one<P, NE, false, EPI, 1>(A, bs, s);
  return 0;
}

template <int P, int NE>
inline int launch_epi(const WilsonArgs& A, int nr, int bs, hipStream_t s) {
  switch (A.epi) {
    case EPI_HOP: return launch_nr<P, NE, EPI_HOP>(A, nr, bs, s);
    case EPI_XPAY: return launch_nr<P, NE, EPI_XPAY>(A, nr, bs, s);
    case EPI_XPAY_NORM:
      if (A.dag) return -1;
      return launch_nr<P, NE, EPI_XPAY_NORM>(A, nr, bs, s);
    case EPI_XPAY_G5: return launch_nr<P, NE, EPI_XPAY_G5>(A, nr, bs, s);
    case EPI_CHEB: return launch_nr<P, NE, EPI_CHEB>(A, nr, bs, s);
    default: break;
  }
  if constexpr (P != 16) {
    switch (A.epi) {
      case EPI_CLOVINV: return launch_nr<P, NE, EPI_CLOVINV>(A, nr, bs, s);
      case EPI_XMY_CLOVINV: return launch_nr<P, NE, EPI_XMY_CLOVINV>(A, nr, bs, s);
      case EPI_XMY_RTS: return launch_nr<P, NE, EPI_XMY_RTS>(A, nr, bs, s);
      case EPI_CLOVINV_XPAY: return launch_nr<P, NE, EPI_CLOVINV_XPAY>(A, nr, bs, s);
      case EPI_SITE: return launch_nr<P, NE, EPI_SITE>(A, nr, bs, s);
      default: break;
    }
  }
  if constexpr (P == 32) {  // the multigrid cycle's
    if (A.dag) return -1;
    if (A.epi == EPI_RESID) return launch_nr<P, NE, EPI_RESID>(A, nr, bs, s);
    if (A.epi == EPI_CLOVINV_ACC) return launch_nr<P, NE, EPI_CLOVINV_ACC>(A, nr, bs, s);
  }
  return -1;
}

template <int P>
int launch_wilson_prec(const WilsonArgs& A, int nr, int bs, hipStream_t s) {
  if constexpr (P != 64) {
    if (A.recon) return launch_epi<P, 6>(A, nr, bs, s);
  }
  return launch_epi<P, 9>(A, nr, bs, s);
}

}  // namespace lq
