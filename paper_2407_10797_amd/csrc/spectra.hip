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
// |B - beta_q| <= 1 / (2 Q) alone: with |e_j| half an ulp of f, up to 3.4e-12 rad at 2.5
// years, Q = 512 and 62.5-125 mHz, and 2.7e-11 with Q = 64.  spec_fmax (fstat_kernels.hip)
// keeps the FP64 block loop to frequencies where that is within the refinement budget.
//
// Why 16 nodes, Q = 2 L (FP64) and Q = L (FP32): over a half block the remaining slope turns
// g by at most pi / 4 (Q = 2 L) and the curvature by kSpecPsiFp64 = 0.25 rad; the
// interpolant of e^{i (0.785 x + 0.25 x^2)} then misses a bin by at most 1.5e-13 (rms
// 1e-13; computed for L = 32 to 256).  With Q = L the slope turns it by pi / 2 and the
// curvature may reach 1 rad, where the largest error is 1.0e-8 (rms 6e-9), below the mixed
// path's FP32 resolution.  16 nodes of 8 + 8 bytes (real and
// imaginary part side by side: one load per lane) are two whole 128-byte lines per
// (block, slope) row.
//
// Measured at 4096 particles x 64 partitions on 7,101,001 bins: the bin sums take 1.16 ms
// (whole blocks) + 0.49 ms (partial ones) instead of 6.8 ms in FP64, 0.80 + 0.30 instead of
// 3.3 ms mixed; the largest partition error against the exact loop is unchanged
// (2.6e-12, 2.1e-11, 2.3e-10 at Np = 1, 64, 256).
#include <cmath>
#include <type_traits>

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

// The weights of every block size: constants of the node positions, so that a plan neither
// forms nor uploads them (0.1 ms of a plan of 180,001 bins).  Block size L from row
// lag_row(L) on: 16 + 32 + 64 + 128 rows.
__constant__ double c_lag[240 * kSpecNodes];
constexpr int lag_row(int L) { return L / 2 - 16; }

// Half sums and differences of the Lagrange polynomials of mirrored nodes at the bins of the
// block's right half: [pair p][0..7] (l_m + l_{15-m}) / 2, [8..15] (l_m - l_{15-m}) / 2 at
// bin c + p + 1/2 (long double on the host; nodes x_m = cos(pi (m + 1/2) / 16), x = y / c).
static void spectra_weights(int32_t L, double* out) {
  const long double pi = 3.141592653589793238462643383279502884L;
  const int M = kSpecNodes;
  long double xm[kSpecNodes];
  for (int m = 0; m < M; ++m) xm[m] = cosl(pi * (m + 0.5L) / M);
  // l_m(x) = c_m prod_{k < m} (x - x_k) prod_{k > m} (x - x_k), the products shared by
  // all m (48 products per bin for 240 quotients: 0.11 ms of a plan's 3.24)
  long double cm[kSpecNodes];
  for (int m = 0; m < M; ++m) {
    cm[m] = 1.0L;
    for (int k = 0; k < M; ++k)
      if (k != m) cm[m] *= xm[m] - xm[k];
    cm[m] = 1.0L / cm[m];
  }
  for (int p = 0; p < L / 2; ++p) {
    const long double x = (p + 0.5L) / ((L - 1) * 0.5L);
    long double l[kSpecNodes], r = 1.0L;
    for (int m = 0; m < M; ++m) {
      l[m] = cm[m] * r;
      r *= x - xm[m];
    }
    r = 1.0L;
    for (int m = M - 1; m >= 0; --m) {
      l[m] *= r;
      r *= x - xm[m];
    }
    for (int m = 0; m < kHalf; ++m) {
      out[p * M + m] = (double)(0.5L * (l[m] + l[M - 1 - m]));
      out[p * M + kHalf + m] = (double)(0.5L * (l[m] - l[M - 1 - m]));
    }
  }
}

int spectra_tables_init() {
  double h[240 * kSpecNodes];
  for (int L = 32; L <= 256; L *= 2) spectra_weights(L, h + lag_row(L) * kSpecNodes);
  return hipMemcpyToSymbol(HIP_SYMBOL(c_lag), h, sizeof(h)) == hipSuccess ? 0 : -1;
}

// One thread per slope of a block (the block index, w and the Lagrange weights are the same
// for the whole wavefront: scalar loads).  Bins are taken in mirrored pairs t = c +- (p + 1/2):
// l_m(-x) = l_{15-m}(x), so the sums and differences of a pair serve two nodes each, 16 FMAs
// per bin instead of 32.  Bound by FP64 issue: about 27 instructions per bin and slope.
template <typename T>
__global__ __launch_bounds__(64) void k_spectra(Grid g, const double* __restrict__ wr,
                                                 const double* __restrict__ wi, int L, int Q,
                                                 int nslots, int nblk, int q0,
                                                 T* __restrict__ S) {
  typedef typename std::conditional<sizeof(T) == 8, double2, float2>::type T2;
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
  const double* lag = c_lag + lag_row(L) * kSpecNodes;
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
  T2* o = reinterpret_cast<T2*>(S) + ((int64_t)b * nslots + q) * kSpecNodes;
#pragma unroll
  for (int m = 0; m < kHalf; ++m) {
    o[m] = T2{(T)(Er[m] + Or[m]), (T)(Ei[m] + Oi[m])};
    o[kSpecNodes - 1 - m] = T2{(T)(Er[m] - Or[m]), (T)(Ei[m] - Oi[m])};
  }
}

// The same rows for Q = 512 slopes on blocks of 256 bins by transforms of length 512 over
// the bins (the upper half zero), one per node: with W = w l_m and W' = w l_m e,
//   S[q][m] = e^{-2 pi i q c / Q} (F[q mod Q] - i (2 pi q / (Q df)) F'[q mod Q]),
// F, F' the transforms of W and W' (the grid term in first order, as above).  A work group
// of 512 threads takes eight nodes of a block (sixteen in 1024 threads would leave 128
// registers for the ~220 in use): thread (j, m) has eight of node m's values in each of
// three radix-8 stages, which exchange through LDS as [value][node], so that LDS accesses
// and the rows' stores are whole 128-byte lines (64 in FP32).  Twiddles come from a table of 1024 roots in LDS; a
// thread's four weights l_m stay in its registers over the blocks that its group takes.
// About 1/6 of the direct sums' operations: 6.3 -> 1.83 ms on 7,101,001 bins, both tables
// (4.5 GB, so 2.5 TB/s; the barriers between the stages keep it from the rate of a copy).
// Shorter blocks, and Q = L alone, keep the direct sums: their cost falls with Q.
constexpr int kFftQ = 512;
constexpr int kFftNodes = 8;              // nodes per work group: half a row
constexpr int kFftThreads = kFftQ / 8 * kFftNodes;
constexpr int kFftGroups = 512;           // a multiple of 16: pairs of groups on one XCD
static_assert(kSpecMaxSlope * kFftQ + 1.5 < kFftQ + 64, "a thread has one slope past the cycle");

struct Cplx {
  double r, i;
};
__device__ __forceinline__ Cplx cadd(Cplx a, Cplx b) { return {a.r + b.r, a.i + b.i}; }
__device__ __forceinline__ Cplx csub(Cplx a, Cplx b) { return {a.r - b.r, a.i - b.i}; }
__device__ __forceinline__ Cplx cmul(Cplx a, double2 w) {
  return {fma(a.r, w.x, -(a.i * w.y)), fma(a.r, w.y, a.i * w.x)};
}
__device__ __forceinline__ Cplx ci(Cplx a) { return {-a.i, a.r}; }        // i a
// x[k] <- sum_a x[a] e^{2 pi i a k / 8}
__device__ __forceinline__ void dft8(Cplx x[8]) {
  const double h = 0.70710678118654752440;
  Cplx e[4], o[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    e[a] = cadd(x[a], x[a + 4]);
    o[a] = csub(x[a], x[a + 4]);
  }
  // odd outputs: o[a] e^{2 pi i a / 8}
  o[1] = Cplx{(o[1].r - o[1].i) * h, (o[1].r + o[1].i) * h};
  o[2] = ci(o[2]);
  o[3] = Cplx{(-o[3].r - o[3].i) * h, (o[3].r - o[3].i) * h};
  auto dft4 = [](const Cplx y[4], Cplx& k0, Cplx& k1, Cplx& k2, Cplx& k3) {
    const Cplx s = cadd(y[0], y[2]), d = csub(y[0], y[2]);
    const Cplx t = cadd(y[1], y[3]), u = ci(csub(y[1], y[3]));
    k0 = cadd(s, t);
    k1 = cadd(d, u);
    k2 = csub(s, t);
    k3 = csub(d, u);
  };
  dft4(e, x[0], x[2], x[4], x[6]);
  dft4(o, x[1], x[3], x[5], x[7]);
}

// Values x[a] at 64 a + j (j this thread's) of node m (0 .. 7) -> transform at j + 64 k, k the index.
__device__ __forceinline__ void fft512(Cplx x[8], int j, int m, double2* buf, const double2* root) {
  dft8(x);
  __syncthreads();                          // the last transform's reads are done
#pragma unroll
  for (int k = 0; k < 8; ++k) {             // [k0][j]
    const Cplx v = k ? cmul(x[k], root[2 * ((j * k) & (kFftQ - 1))]) : x[k];
    buf[(k * 64 + j) * kFftNodes + m] = double2{v.r, v.i};
  }
  __syncthreads();
  const int k0 = j >> 3, c = j & 7;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const double2 v = buf[(k0 * 64 + b * 8 + c) * kFftNodes + m];
    x[b] = Cplx{v.x, v.y};
  }
  dft8(x);
#pragma unroll
  for (int k = 0; k < 8; ++k) {             // [k0][k1][c], over what this thread read
    const Cplx v = k ? cmul(x[k], root[16 * c * k]) : x[k];
    buf[(k0 * 64 + k * 8 + c) * kFftNodes + m] = double2{v.r, v.i};
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 8; ++e) {             // now k0 = j % 8, k1 = j / 8
    const double2 v = buf[((j & 7) * 64 + (j >> 3) * 8 + e) * kFftNodes + m];
    x[e] = Cplx{v.x, v.y};
  }
  dft8(x);
}

template <bool D32>
__global__ __launch_bounds__(kFftThreads) void k_spectra_fft(Grid g, const double* __restrict__ wr,
                                                             const double* __restrict__ wi,
                                                             int nslots, int n32, int nblk,
                                                             double* __restrict__ s64,
                                                             float* __restrict__ s32) {
  extern __shared__ double2 s_fft[];
  double2* buf = s_fft;                                  // [512][8]
  double2* root = s_fft + kFftQ * kFftNodes;            // e^{2 pi i k / 1024}
  constexpr int L = kFftQ / 2;
  const int m = threadIdx.x & (kFftNodes - 1), j = threadIdx.x / kFftNodes;
  // groups 16 i + x and 16 i + 8 + x (one XCD) take the two halves of a block's rows
  const int node = m + kFftNodes * ((blockIdx.x >> 3) & 1);
  const int first = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7), step = gridDim.x / 2;
  for (int k = threadIdx.x; k < 2 * kFftQ; k += kFftThreads) {
    double s, c;
    sincospi((double)k / (double)kFftQ, &s, &c);
    root[k] = double2{c, s};
  }
  const double* lag = c_lag + lag_row(L) * kSpecNodes;
  // l_m at bins 64 a + j: the half sums and differences at the bin's mirrored pair
  double lm[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int t = 64 * a + j, pr = t >= L / 2 ? t - L / 2 : L / 2 - 1 - t;
    const int mm = min(node, kSpecNodes - 1 - node);
    const double E = lag[pr * kSpecNodes + mm], O = lag[pr * kSpecNodes + kHalf + mm];
    lm[a] = (node < kHalf) == (t >= L / 2) ? E + O : E - O;
  }
  const double kap = 6.283185307179586477 / (double)kFftQ / g.df;
  for (int b = first; b < nblk; b += step) {
    const int64_t j0 = (int64_t)b * L;
    Cplx x[8], y[8];
    const Cplx zero{0.0, 0.0};
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int64_t jj = j0 + 64 * a + j;
      x[a] = Cplx{wr[jj] * lm[a], wi[jj] * lm[a]};
      x[a + 4] = zero;
    }
    fft512(x, j, m, buf, root);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int64_t jj = j0 + 64 * a + j;
      const double d = (double)(g.k_lo + jj);
      const double e = lm[a] * fma(d, g.df, -(d * g.df));
      y[a] = Cplx{wr[jj] * e, wi[jj] * e};
      y[a + 4] = zero;
    }
    fft512(y, j, m, buf, root);
    double2* o64 = reinterpret_cast<double2*>(s64) + (int64_t)b * nslots * kSpecNodes + node;
    float2* o32 = reinterpret_cast<float2*>(s32) + (int64_t)b * n32 * kSpecNodes + node;
    auto put = [&](int q, Cplx f, Cplx fe) {
      if (q >= nslots) return;
      const double k = kap * (double)q;
      const Cplx v = cmul(Cplx{fma(k, fe.i, f.r), fma(-k, fe.r, f.i)},
                          root[(2 * kFftQ - (2 * (L / 2) - 1) * q) & (2 * kFftQ - 1)]);
      o64[(int64_t)q * kSpecNodes] = double2{v.r, v.i};
      if (D32 && !(q & 1) && (q >> 1) < n32) {
        o32[(int64_t)(q >> 1) * kSpecNodes] = float2{(float)v.r, (float)v.i};
      }
    };
#pragma unroll
    for (int k = 0; k < 8; ++k) put(j + 64 * k, x[k], y[k]);
    put(j + kFftQ, x[0], y[0]);              // slopes of a whole cycle per bin and above
  }
}

template <typename T>
static void launch_direct(const Grid& g, const double* wr, const double* wi,
                          const Spectra<T>& t, T* S, hipStream_t s) {
  // slopes in whole wavefronts per block, then the few left over (the last one of Q + 1)
  // with the blocks across the lanes
  const int bs = 64, whole = t.nslots / bs;
  if (whole > 0)
    hipLaunchKernelGGL(k_spectra<T>, dim3(t.nblk, whole), dim3(bs), 0, s, g, wr, wi, t.L, t.Q,
                       t.nslots, t.nblk, -1, S);
  for (int q = whole * bs; q < t.nslots; ++q)
    hipLaunchKernelGGL(k_spectra<T>, dim3((t.nblk + bs - 1) / bs), dim3(bs), 0, s, g, wr, wi, t.L,
                       t.Q, t.nslots, t.nblk, q, S);
}

// With both tables their blocks are of 256 bins (spectra_block), which the transforms take.
void launch_spectra(const Grid& g, const double* wr, const double* wi,
                    const Spectra<double>& t64, const Spectra<float>& t32, double* s64, float* s32,
                    hipStream_t s) {
  if (!s64) {
    launch_direct(g, wr, wi, t32, s32, s);
  } else if (t64.Q == kFftQ && t64.L == kFftQ / 2) {
    auto fft = s32 ? k_spectra_fft<true> : k_spectra_fft<false>;
    const size_t lds = sizeof(double2) * (kFftQ * kFftNodes + 2 * kFftQ);
    (void)hipFuncSetAttribute((const void*)fft, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    hipLaunchKernelGGL(fft, dim3(kFftGroups), dim3(kFftThreads), lds, s, g, wr, wi,
                       t64.nslots, t32.nslots, t64.nblk, s64, s32);
  } else {
    launch_direct(g, wr, wi, t64, s64, s);
  }
}

}  // namespace fstat
