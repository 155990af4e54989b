// Wilson-type stencil dispatcher (FP64 instantiations) and the site-term
// kernel of the twisted-clover operator.  The stencil templates live in
// wilson_impl.h; FP32 and FP16 instantiations are in wilson32.hip and
// wilson16.hip so that the three precisions compile in parallel.
#include "wilson_impl.h"

namespace lq {

template int launch_wilson_prec<64>(const WilsonArgs& A, int nr, int bs, hipStream_t s);
extern template int launch_wilson_prec<32>(const WilsonArgs& A, int nr, int bs, hipStream_t s);
extern template int launch_wilson_prec<16>(const WilsonArgs& A, int nr, int bs, hipStream_t s);

int launch_wilson(const WilsonArgs& A, hipStream_t s) {
  if (A.prec == 16 && (A.epi == EPI_CLOVINV || A.epi == EPI_XMY_CLOVINV || A.epi == EPI_SITE ||
                       A.epi == EPI_XMY_RTS || A.epi == EPI_CLOVINV_XPAY || A.epi == EPI_RESID ||
                       A.epi == EPI_CLOVINV_ACC))
    return -1;
  const int nr = A.nr > 0 || A.nr == kSplitShape ? A.nr : 1;
  if (!traversal_valid(A.g, A.slab)) return -1;
  const int bs = 0;
  int r;
  if (A.prec == 64) r = launch_wilson_prec<64>(A, nr, bs, s);
  else if (A.prec == 32) r = launch_wilson_prec<32>(A, nr, bs, s);
  else r = launch_wilson_prec<16>(A, nr, bs, s);
  if (r) return r;
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace lq

namespace lq {

// Site term (clover + twist) applied alone: out = A x or A^{-1} x per site.
// Bound by HBM; a thread takes a site and KC columns, so that the matrix (A 288 B,
// A^{-1} 576 B per site in FP32) is read once per KC columns.
template <int P, bool INV, int KC>
__global__ void __launch_bounds__(256) site_kernel(Geom g, const void* clov, const void* clov_inv, double mu_tw,
                                                   FieldRef in, FieldRef out, int par_out, int ncol) {
  using R = typename RealOf<P>::T;
  const int nsite = par_out == 2 ? 2 * g.Vh : g.Vh;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= nsite) return;
  const int col0 = blockIdx.y * KC, nv = min(KC, ncol - col0);
  const int par = par_out == 2 ? (j >= g.Vh) : par_out;
  const int cb = par_out == 2 ? j - par * g.Vh : j;
  cx<R> x[KC][12];
#pragma unroll
  for (int r = 0; r < KC; ++r)
    if (r < nv) IO<P, 12>::load(in, blk_index(in, col0 + r, par), cb, x[r]);
  if constexpr (INV) {
    apply_full6_nr<P, KC>(clov_inv, g.Vh, par, 0, cb, nv, x, 0);
    apply_full6_nr<P, KC>(clov_inv, g.Vh, par, 1, cb, nv, x, 6);
  }
#pragma unroll
  for (int r = 0; r < KC; ++r) {
    if (r >= nv) continue;
    if constexpr (INV) {
      IO<P, 12>::store(out, blk_index(out, col0 + r, par), cb, x[r]);
    } else {
      cx<R> y[12];
      apply_herm6<P>(clov, g.Vh, par, 0, cb, x[r], y);
      apply_herm6<P>(clov, g.Vh, par, 1, cb, x[r] + 6, y + 6);
      const R mu = (R)mu_tw;
#pragma unroll
      for (int k = 0; k < 6; ++k) y[k] = y[k] + mu * times_i(x[r][k]);
#pragma unroll
      for (int k = 6; k < 12; ++k) y[k] = y[k] - mu * times_i(x[r][k]);
      IO<P, 12>::store(out, blk_index(out, col0 + r, par), cb, y);
    }
  }
}

// Columns per thread.  Four cost registers (A^{-1} in FP64 spills 228 B per lane
// and is still the fastest from three columns), which fewer columns pay for
// without a use.  Times in us with 1 / 2 / 4 columns per thread:
//   A^{-1} FP64 16^3x32  1 column 33 / 33 / 37, 3: 96 / 78 / 68, 12: 304 / 248 / 249
//               24^3x64  1: 279 / 274 / 300, 3: 819 / 588 / 407, 12: 3189 / 1932 / 1509
//   A^{-1} FP32 24^3x64  1: 148 / 127 / 130, 3: 428 / 287 / 187, 12: 1618 / 959 / 652
//   A      FP32 24^3x64  1: 69 / 71 / 71, 3: 226 / 197 / 179, 12: 929 / 700 / 699
//   A      FP64 16^3x32  1: 19 / 21 / 29, 4: 69 / 76 / 89, 12: 197 / 212 / 229
//               20^3x48  1: 76 / 76 / 118, 4: 271 / 247 / 250, 12: 782 / 664 / 651
//               24^3x64  1: 174 / 172 / 274, 4: 646 / 531 / 526, 12: 1933 / 1482 / 1389
// A in FP64 gains nothing from fewer reads while its matrices stay in the last-level
// cache (75 MiB at 16^3x32, 108 at 16^2x24x32; 211 at 20^3x48), and holds 256
// registers with four columns.
static int site_cols(int prec, bool inverse, int nsite, int ncol) {
  if (prec == 64 && !inverse) {
    if ((int64_t)nsite * 576 <= (int64_t)128 << 20) return 1;
    return ncol < 8 ? 2 : 4;
  }
  return ncol <= 2 ? 2 : 4;
}

int launch_site(const Geom& g, int prec, const void* clov, const void* clov_inv, double mu_tw, bool inverse,
                FieldRef in, FieldRef out, int par_out, int ncol, hipStream_t s) {
  const int nsite = par_out == 2 ? 2 * g.Vh : g.Vh;
  if (nsite == 0 || ncol == 0) return 0;
  if (prec != 64 && prec != 32) return -8;
  const int kc = site_cols(prec, inverse, nsite, ncol);
  const dim3 grid((nsite + 255) / 256, (ncol + kc - 1) / kc);
#define LQ_SITE(P, INV, KC)                                   \
  if (prec == P && inverse == INV && kc == KC)                \
    site_kernel<P, INV, KC><<<grid, 256, 0, s>>>(g, clov, clov_inv, mu_tw, in, out, par_out, ncol);
  LQ_SITE(64, false, 1) LQ_SITE(64, false, 2) LQ_SITE(64, false, 4) LQ_SITE(64, true, 2) LQ_SITE(64, true, 4)
  LQ_SITE(32, false, 2) LQ_SITE(32, false, 4) LQ_SITE(32, true, 2) LQ_SITE(32, true, 4)
#undef LQ_SITE
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

}  // namespace lq
