// spectra.hip -- block spectra of a plan's data.
//
// The N-terms of an item are sums over bins of w_j e^{i Phi_j} T(s_j).  Within a block of L
// bins the phase is a straight line of slope B = dPhi/dj (about t_f df cycles per bin, in
// [0, T_obs df]) plus a curvature of a fraction of a radian, so with a slope beta_q = q / Q
// near B the factor g(t) = e^{i (Phi - 2 pi beta_q t)} T(s) is a smooth function of the bin:
// a polynomial in t through kSpecNodes Chebyshev points reproduces it, and
//   sum_t w_t e^{i Phi_t} T_t = sum_m g(y_m) S[q][m],
//   S[q][m] = sum_t w_t e^{2 pi i beta_q (t - c)} l_m(t)
// with l_m the Lagrange polynomials of the nodes, c = (L - 1) / 2 the block's centre and
// t - c = y_m the node positions.  S does not depend on the template: it is the data, laid
// out once per plan, and an item then costs kSpecNodes samples per block instead of L.
//
// The grid is f_j = (k_lo + j) df rounded to a double; e_j = exact - rounded.  The slope's
// phase is taken at the rounded frequency, e^{2 pi i beta_q ((t - c) - e_j / df)} (the second
// factor to first order: |2 pi beta_q e_j / df| <~ 4e-9), which leaves the grid term of
// |B - beta_q| <= 1 / (2 Q) alone, below 2e-12 rad at 2.5 years.
//
// Why 16 nodes, Q = 2 L (FP64) and Q = L (FP32): over a half block the remaining slope turns
// g by at most pi / 4 (Q = 2 L) and the curvature by kSpecPsi64 = 0.25 rad; the Chebyshev
// coefficients of e^{i (0.785 x + 0.25 x^2)} fall below 1e-13 at degree 16.  With Q = L the
// slope turns it by pi / 2 and the curvature may reach 1 rad before the sixteenth coefficient
// passes 1e-8, the mixed path's FP32 resolution.  16 nodes of 8 + 8 bytes are two whole
// 128-byte lines per (block, slope) row.
//
// Measured at 4096 particles x 64 partitions on 7,101,001 bins: the bin sums take 1.31 ms
// (whole blocks) + 0.50 ms (partial ones) instead of 6.8 ms in FP64, 0.82 + 0.30 instead of
// 3.3 ms mixed; the largest partition error against the exact loop is unchanged
// (2.6e-12, 2.1e-11, 2.3e-10 at Np = 1, 64, 256).
#include <cmath>

#include "fstat_kernels.h"

namespace fstat {

constexpr int kHalf = kSpecNodes / 2;

// Largest block for which the curvature of the data set's templates stays inside the bound:
// the second difference of the phase is about 1 / (support bins) cycles per bin^2 and at most
// ~30 / nbins over the parameter ranges of the searches (measured: 28 / nbins for chirp masses
// 10-50 at 7.1e6 bins), so psi = pi (30 / nbins) (L / 2)^2 <= 0.25 (FP64) or 1 (FP32).
// Items that exceed the bound all the same take the per-bin loop.  Below 32 bins a block
// saves too little: those data sets have no spectra.  256 bins suffice where longer blocks
// would still pass: the partial blocks at a partition's ends are evaluated bin by bin, and
// with longer blocks they outweigh the whole ones.
int spectra_block(bool mixed, int64_t nbins) {
  const double L = (mixed ? 0.206 : 0.103) * std::sqrt((double)nbins);
  int b = 256;
  while (b >= 32 && (double)b > L) b >>= 1;
  return b >= 32 ? b : 0;
}

int spectra_slots(const Grid& g, int32_t Q) {
  return (int)std::floor(g.T_obs * g.df * (double)Q + 0.5) + 1;
}

// Half sums and differences of the Lagrange polynomials of mirrored nodes at the bins of the
// block's right half: [pair p][0..7] (l_m + l_{15-m}) / 2, [8..15] (l_m - l_{15-m}) / 2 at
// bin c + p + 1/2 (long double on the host; nodes x_m = cos(pi (m + 1/2) / 16), x = y / c).
void spectra_weights(int32_t L, double* out) {
  const long double pi = 3.141592653589793238462643383279502884L;
  const int M = kSpecNodes;
  long double xm[kSpecNodes];
  for (int m = 0; m < M; ++m) xm[m] = cosl(pi * (m + 0.5L) / M);
  for (int p = 0; p < L / 2; ++p) {
    const long double x = (p + 0.5L) / ((L - 1) * 0.5L);
    long double l[kSpecNodes];
    for (int m = 0; m < M; ++m) {
      l[m] = 1.0L;
      for (int k = 0; k < M; ++k)
        if (k != m) l[m] *= (x - xm[k]) / (xm[m] - xm[k]);
    }
    for (int m = 0; m < kHalf; ++m) {
      out[p * M + m] = (double)(0.5L * (l[m] + l[M - 1 - m]));
      out[p * M + kHalf + m] = (double)(0.5L * (l[m] - l[M - 1 - m]));
    }
  }
}

// One thread per slope of a block (the block index, w and the Lagrange weights are the same
// for the whole wavefront: scalar loads).  Bins are taken in mirrored pairs t = c +- (p + 1/2):
// l_m(-x) = l_{15-m}(x), so the sums and differences of a pair serve two nodes each, 16 FMAs
// per bin instead of 32.  Bound by FP64 issue: about 27 instructions per bin and slope.
template <bool D64, bool D32>
__global__ __launch_bounds__(64) void k_spectra(Grid g, const double* __restrict__ wr,
                                                 const double* __restrict__ wi, int L, int Q,
                                                 int nslots, int n32, int nblk, int q0,
                                                 const double* __restrict__ lag,
                                                 double* __restrict__ s64,
                                                 float* __restrict__ s32) {
  const int q = q0 >= 0 ? q0 : blockIdx.y * blockDim.x + threadIdx.x;
  const int b = q0 >= 0 ? blockIdx.x * blockDim.x + threadIdx.x : blockIdx.x;
  if (q >= nslots || b >= nblk) return;
  const int64_t j0 = (int64_t)b * L;
  const double beta = (double)q / (double)Q;
  const double kap = 6.283185307179586477 * beta / g.df;
  double zr, zi, er, ei;                       // z = e^{2 pi i beta}, (er, ei) = z^{p + 1/2}
  sincospi(2.0 * beta, &zi, &zr);
  sincospi(beta, &ei, &er);
  double Er[kHalf], Ei[kHalf], Or[kHalf], Oi[kHalf];
#pragma unroll
  for (int m = 0; m < kHalf; ++m) Er[m] = Ei[m] = Or[m] = Oi[m] = 0.0;
  const int half = L >> 1;
  for (int p = 0; p < half; ++p) {
    const int64_t jr = j0 + half + p, jl = j0 + half - 1 - p;
    const double dr = (double)(g.k_lo + jr), dl = (double)(g.k_lo + jl);
    const double xr = -kap * fma(dr, g.df, -(dr * g.df));   // grid term of each bin
    const double xl = -kap * fma(dl, g.df, -(dl * g.df));
    const double a0 = wr[jr], a1 = wi[jr], b0 = wr[jl], b1 = wi[jl];
    const double ar = fma(-xr, a1, a0), ai = fma(xr, a0, a1);
    const double br = fma(-xl, b1, b0), bi = fma(xl, b0, b1);
    // right bin times z^{p + 1/2}, left bin times its conjugate
    const double Rr = fma(ar, er, -(ai * ei)), Ri = fma(ar, ei, ai * er);
    const double Lr = fma(br, er, bi * ei), Li = fma(-br, ei, bi * er);
    const double ur = Rr + Lr, ui = Ri + Li, vr = Rr - Lr, vi = Ri - Li;
    const double* lp = lag + p * kSpecNodes;
#pragma unroll
    for (int m = 0; m < kHalf; ++m) {
      Er[m] = fma(lp[m], ur, Er[m]);
      Ei[m] = fma(lp[m], ui, Ei[m]);
      Or[m] = fma(lp[kHalf + m], vr, Or[m]);
      Oi[m] = fma(lp[kHalf + m], vi, Oi[m]);
    }
    const double nr = fma(er, zr, -(ei * zi));
    ei = fma(er, zi, ei * zr);
    er = nr;
  }
  if constexpr (D64) {
    double* o = s64 + ((int64_t)b * nslots + q) * (2 * kSpecNodes);
#pragma unroll
    for (int m = 0; m < kHalf; ++m) {
      o[m] = Er[m] + Or[m];
      o[kSpecNodes - 1 - m] = Er[m] - Or[m];
      o[kSpecNodes + m] = Ei[m] + Oi[m];
      o[2 * kSpecNodes - 1 - m] = Ei[m] - Oi[m];
    }
  }
  if constexpr (D32) {
    // with both tables the FP32 one keeps every second slope (Q = L beside Q = 2 L)
    const int q32 = D64 ? q >> 1 : q;
    if (!D64 || ((q & 1) == 0 && q32 < n32)) {
      float* o = s32 + ((int64_t)b * n32 + q32) * (2 * kSpecNodes);
#pragma unroll
      for (int m = 0; m < kHalf; ++m) {
        o[m] = (float)(Er[m] + Or[m]);
        o[kSpecNodes - 1 - m] = (float)(Er[m] - Or[m]);
        o[kSpecNodes + m] = (float)(Ei[m] + Oi[m]);
        o[2 * kSpecNodes - 1 - m] = (float)(Ei[m] - Oi[m]);
      }
    }
  }
}

void launch_spectra(const Grid& g, const double* wr, const double* wi, const double* lag,
                    const Spectra<double>& t64, const Spectra<float>& t32, double* s64, float* s32,
                    hipStream_t s) {
  const int L = s64 ? t64.L : t32.L, Q = s64 ? t64.Q : t32.Q;
  const int ns = s64 ? t64.nslots : t32.nslots, nblk = s64 ? t64.nblk : t32.nblk;
  auto kern = s64 ? (s32 ? k_spectra<true, true> : k_spectra<true, false>)
                  : k_spectra<false, true>;
  // slopes in whole wavefronts per block, then the few left over (the last one of Q + 1)
  // with the blocks across the lanes
  const int bs = 64, whole = ns / bs;
  if (whole > 0)
    hipLaunchKernelGGL(kern, dim3(nblk, whole), dim3(bs), 0, s, g, wr, wi, L, Q, ns, t32.nslots,
                       nblk, -1, lag, s64, s32);
  for (int q = whole * bs; q < ns; ++q)
    hipLaunchKernelGGL(kern, dim3((nblk + bs - 1) / bs), dim3(bs), 0, s, g, wr, wi, L, Q, ns,
                       t32.nslots, nblk, q, lag, s64, s32);
}

}  // namespace fstat
