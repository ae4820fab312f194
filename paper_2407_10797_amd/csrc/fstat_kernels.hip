// fstat_kernels.hip -- gfx950 kernels of the batched semi-coherent F-statistic.
//
// One evaluation (Sec. II.B, Eq. semi-cohF of arXiv:2407.10797) is a chain of
// kernels:
//   k_setup         one wavefront per particle: intrinsic parameters -> PN
//                   constants, sky frame, support [f_lo, f_hi] (t_f inverted by
//                   two clustered searches), Np partition edges (bin indices) and the
//                   work-item counts: a work item is the part of a partition inside
//                   one tile of the global tiling of the band, or a few tiles
//   k_worklist      exclusive scan of the work-item counts and the work list, item
//                   -> (particle*stride + partition, tile and tiles); for many
//                   particles k_scan_* (three passes) and k_fill
//   k_interp_nodes  exact template at 10 Chebyshev nodes and both ends of every
//                   item -> interpolation record, or hand-over to the exact loop;
//                   the M-terms by quadrature
//   k_tile_*        items grouped by tile, the block loop's and the per-bin loop's
//                   (k_tile_group: small calls, in one block)
//   k_eval_blocks   N-terms of whole blocks from the plan's block spectra
//                   (spectra.hip): sixteen samples per block
//   k_eval_edges    N-terms of the partial blocks at a partition's ends, bin by bin
//   k_eval_interp   the per-bin loop, for items without block spectra: persistent
//                   blocks take scheduling units of <= 64 items of a tile, stage the
//                   tile's data in LDS, and evaluate the interpolated template at
//                   every bin (FP64: advanced by a difference recurrence along each
//                   lane's run of bins); deterministic sums, no float atomics
//   k_eval_exact    the exact template at every bin, for handed-over items, for
//                   refinement and under FSTAT_EVAL_EXACT (FP64 and mixed)
//   k_mark          partitions whose interpolation error could matter -> exact
//   k_solve         eight lanes per (particle, partition): ordered sum of the
//                   item partials and the 2x2 Hermitian closed form of F_l; then
//                   F_hat = mean_l F_l, or -inf / NaN
#include "fstat_internal.h"
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "fstat_kernels.h"
#include "philox.h"

namespace fstat {

// ---------------------------------------------------------------------------
// plan-time per-bin preparation
// ---------------------------------------------------------------------------
// C(f) = (1 - z^2)(-i pi f L) exp(-i pi f L), z = exp(-2 i pi f L): the part of
// the TDI-X transfer shared by every template.  With g = f^{-7/6} e^{-i Psi}
// (App. A) and <a,b> = 4 df Re sum a conj(b) / S (Sec. II.A):
//   w_j = 4 df s_j conj(C_j) f_j^{-7/6} / S_j,   u_j = 4 df |C_j|^2 f_j^{-7/3} / S_j.
__global__ void k_prep(Grid g, const double* __restrict__ data, const double* __restrict__ psd,
                       double* __restrict__ wr, double* __restrict__ wi, double* __restrict__ u,
                       double* __restrict__ s0, double* __restrict__ c0) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= g.nbins) return;
  const int64_t jc = (int64_t)blockIdx.y * g.nbins + j;   // channel blockIdx.y
  double f = (double)(g.k_lo + j) * g.df;
  double s, c;
  sincospi(kLs * f, &s, &c);
  double x0 = kPi * kLs * f;
  double zr = c * c - s * s, zi = -2.0 * s * c;
  double omr = 1.0 - (zr * zr - zi * zi), omi = -2.0 * zr * zi;  // 1 - z^2
  double er = -x0 * s, ei = -x0 * c;                               // -i x0 e^{-i x0}
  double Cr = omr * er - omi * ei, Ci = omr * ei + omi * er;
  double amp = pow(f, -7.0 / 6.0);
  double wgt = 4.0 * g.df / psd[jc];
  double dr = data[2 * jc], di = data[2 * jc + 1];
  // s conj(C)
  double pr = dr * Cr + di * Ci, pi = di * Cr - dr * Ci;
  wr[jc] = wgt * amp * pr;
  wi[jc] = wgt * amp * pi;
  u[jc] = wgt * amp * amp * (Cr * Cr + Ci * Ci);
  if (blockIdx.y == 0) {
    s0[j] = s;
    c0[j] = c;
  }
}

__global__ void k_zero64(unsigned long long* __restrict__ x) {
  if (threadIdx.x == 0) x[0] = 0ull;
}

// max of u over the band -> *out (zero before): u > 0, so the order of the
// doubles is that of their bits.  One atomic per block, and blocks for the bins there
// are: an atomic from each of 4096 wavefronts took 48 us whatever the band (a plan of
// 20,972 bins 0.105 -> 0.149 ms).
__global__ __launch_bounds__(256) void k_max(const double* __restrict__ u, int64_t n,
                                             unsigned long long* __restrict__ out) {
  __shared__ double red[4];
  double m = 0.0;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * blockDim.x)
    m = fmax(m, u[j]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    atomicMax(out, (unsigned long long)__double_as_longlong(m));
  }
}

// Normalise so that max u = 1: F is invariant under (w, u) -> (g w, g^2 u)
// (a rescaling of the template), and FP32 copies stay in range.
__global__ void k_scale(Grid g, const double* __restrict__ umax, double* __restrict__ wr,
                        double* __restrict__ wi, double* __restrict__ u,
                        const double* __restrict__ s0, const double* __restrict__ c0,
                        float* __restrict__ wr32, float* __restrict__ wi32,
                        float* __restrict__ u32, float* __restrict__ s032,
                        float* __restrict__ c032) {
  int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= g.nbins) return;
  const int64_t jc = (int64_t)blockIdx.y * g.nbins + j;   // channel blockIdx.y
  double m = umax[0];
  double gam2 = (m > 0.0) ? 1.0 / m : 1.0;
  double gam = sqrt(gam2);
  double a = wr[jc] * gam, b = wi[jc] * gam, c = u[jc] * gam2;
  wr[jc] = a; wi[jc] = b; u[jc] = c;
  if (wr32) {
    wr32[jc] = (float)a; wi32[jc] = (float)b; u32[jc] = (float)c;
    if (blockIdx.y == 0) { s032[j] = (float)s0[j]; c032[j] = (float)c0[j]; }
  }
}

// ---------------------------------------------------------------------------
// particle setup: constants, support, partition boundaries, work counts
// ---------------------------------------------------------------------------
__device__ __forceinline__ double bin_freq(const Grid& g, int64_t j) {
  return (double)(g.k_lo + j) * g.df;
}

// a / n for 0 <= a < 2^31 and n >= 1 from rn = 1 / n: (a + 1/2) / n is at least
// 1 / (2 n) from a whole number, the product's error below 2^-20 of that (4
// operations; an integer division takes ~25)
__device__ __forceinline__ int div_by(int a, double rn) { return (int)(((double)a + 0.5) * rn); }

// Tiles per work item in a partition.  What an interpolant over an item has to follow
// is the detector's motion (up to four turns a year of the transfer's phase pattern)
// over the time that the signal spends in it, its width times dt/df =
// (5/96) pi^{-8/3} Mc^{-5/3} f^{-11/3}, and the chirp's own shape over width / f.  Both
// fall with f: from tile z on mmax tiles keep the limits, before it the m1 that do at
// the partition's start.  (The first limit with a fifth to spare: 4096 whole-band
// partitions, two swarm iterations, 5.56 ms without z, 4.75, 4.91 and 5.17 with
// factors 1.15, 1.3 and 1.5, but 6.00 with 1, where 6,949 items miss.)  The
// partition's word: z << 3 | m1.
constexpr int kWholeBand = 1 << 27;      // no tile z: beyond any plan's tiles
__device__ __forceinline__ int item_width(const Grid& g, const Tiling& tl, float mc53, int a,
                                          int b) {
  const float f = (float)((double)(g.k_lo + a) * g.df), mx = (float)tl.mmax;
  const float mt = tl.kt * mc53 * powf(f, 11.0f / 3.0f);
  if ((float)(b - a) * (float)tl.rT < tl.kd * mt) return kWholeBand << 3 | 1;
  const int m1 = (int)fminf(fmaxf(fminf(mt, tl.kf * f), 1.0f), mx);
  const double fz = fmaxf(powf(1.2f * mx / (tl.kt * mc53), 3.0f / 11.0f), mx / tl.kf);
  const double z = fmin(fmax(ceil((fz / g.df - (double)g.k_lo) * tl.rT), 0.0), (double)tl.ntiles);
  return ((int)z + tl.mmax - 1) / tl.mmax * tl.mmax << 3 | m1;
}
// Items i of a partition with bins [a, b): n1 of m1 tiles from unit u0 (cut at tile
// z), then those of mmax tiles from unit v0.
struct ItemCut {
  int m1, z, u0, n1, v0;
};
__device__ __forceinline__ int item_count(const Tiling& tl, int a, int b, int word, ItemCut& c) {
  c = ItemCut{1, INT32_MAX, 0, 0, 0};
  if (b <= a) return 0;
  const int ta = div_by(a, tl.rT), tb = div_by(b - 1, tl.rT);
  c.u0 = ta;
  if (tl.mmax == 1) return c.n1 = tb - ta + 1;
  c.m1 = word & 7;
  c.z = word >> 3;
  c.u0 = ta / c.m1;
  c.n1 = ta < c.z ? min(tb, c.z - 1) / c.m1 - c.u0 + 1 : 0;
  c.v0 = max(ta, c.z) / tl.mmax;
  return c.n1 + (tb >= c.z ? tb / tl.mmax - c.v0 + 1 : 0);
}
// A work item: partition q and, in one word, its first tile (the tiles of all
// channels numbered channel by channel) << 3 | its tiles m.  Items of several
// channels: tile by tile, all channels of each.
__device__ __forceinline__ int item_word(int i, const ItemCut& c, const Tiling& tl, int nch) {
  const int ct = nch == 1 ? i : i / nch, ch = i - ct * nch;
  const bool head = ct < c.n1;
  const int t = head ? (c.u0 + ct) * c.m1 : (c.v0 + ct - c.n1) * tl.mmax;
  const int m = head ? min(c.m1, c.z - t) : tl.mmax;
  return (ch * tl.ntiles + t) << 3 | m;
}
__device__ __forceinline__ int item_chan(int y, const Tiling& tl, int nch) {
  return nch > 1 ? (y >> 3) / tl.ntiles : 0;
}
// its bins: those of its tiles that are in the partition's [a, b)
__device__ __forceinline__ void item_bins(int a, int b, int y, int ch, const Tiling& tl, int& b0,
                                          int& b1) {
  const int t = (y >> 3) - ch * tl.ntiles;
  b0 = max(a, t * tl.T);
  b1 = (int)min((int64_t)b, (int64_t)(t + (y & 7)) * tl.T);
}

// smallest j in [lo, hi+1] with f_j >= e
__device__ int first_bin_at_or_above(const Grid& g, double e, int lo, int hi) {
  double jd = ceil(e / g.df) - (double)g.k_lo;
  int j = (jd < (double)lo) ? lo : (jd > (double)(hi + 1) ? hi + 1 : (int)jd);
  while (j > lo && bin_freq(g, j - 1) >= e) --j;
  while (j <= hi && bin_freq(g, j) < e) ++j;
  return j;
}

__device__ double tf_only(const PartConst& P, double f) {
  double fr, tf;
  phase_and_tf(P, f, fr, tf);
  return tf;
}

// Frequencies where t_f (increasing in f) reaches 0 and T_obs on (fa, fb), by
// the two halves of a wavefront (need: this half has a root to find; t_a < t
// and t_b >= t are t_f at the ends).  Each round evaluates 32 points per half
// and the ballot of those below t brackets the root.  The points cluster
// geometrically (factor 8) around a prediction of the root -- first the
// Newtonian chirp's, then the bracket's interpolant, linear in f^{-8/3} (in
// which the Newtonian t_f is linear) while the bracket is wide, linear in f
// after -- so that the bracket shrinks to about eight times the prediction's
// error; a round that gained less than a factor 4, or a bracket of a few
// hundred ulps, is cut evenly.  Ends at two neighbouring doubles; returns the
// upper one.  Six or seven evaluations of t_f in place of the ~40 of two even
// 64-point searches finished by bisection (k_setup 30 -> 15 us for one
// particle, 110 -> 34 us for 4096).
__device__ double invert_tf(const PartConst& P, double t, bool need, double fa, double fb,
                            double ta, double tb, int lane) {
  const int half = lane & 32, i = lane & 31;
  ta -= t;
  tb -= t;
  if (!need) fb = fa;
  double r = 0.5 * (fa + fb);
  {
    const double tau = P.tc - t;
    if (tau > 0.0) {
      const double fn = exp(0.375 * log(5.0 / (256.0 * tau)) - 0.625 * log(P.mc_hi)) * (1.0 / kPi);
      if (fn > fa && fn < fb) r = fn;
    }
  }
  bool even = false;
  const double rho = ldexp(1.0, -3 * (i < 16 ? i + 1 : 32 - i));
  for (int it = 0; it < 64; ++it) {
    const double fm = 0.5 * (fa + fb);
    const bool done = fm <= fa || fm >= fb;
    if (__all(done)) break;
    const double w = fb - fa;
    even = even || w <= 2.3e-13 * fb;
    double f = even ? fa + w * ((double)(i + 1) * (1.0 / 33.0))
                    : (i < 16 ? r - (r - fa) * rho : r + (fb - r) * rho);
    f = fmin(fmax(f, fa), fb);
    const double v = tf_only(P, f) - t;
    const uint32_t below = (uint32_t)(__ballot(v < 0.0) >> half);
    const int k = __popc(below);                   // points below t (a prefix: t_f increases)
    const double f0 = __shfl(f, half + max(k - 1, 0), 64), v0 = __shfl(v, half + max(k - 1, 0), 64);
    const double f1 = __shfl(f, half + min(k, 31), 64), v1 = __shfl(v, half + min(k, 31), 64);
    if (done) continue;                            // shuffles done: this half waits
    if (k > 0) { fa = f0; ta = v0; }
    if (k < 32 && f1 <= fb) { fb = f1; tb = v1; }
    const double w1 = fb - fa;
    even = w1 > 0.25 * w;
    const double x = -ta / (tb - ta);
    if (w1 > 1e-3 * fb) {
      const double la = log(fa), lb = log(fb);
      const double ya = exp((-8.0 / 3.0) * la), yb = exp((-8.0 / 3.0) * lb);
      r = exp(-0.375 * log(fma(x, yb - ya, ya)));
    } else {
      r = fma(x, w1, fa);
    }
    if (!(r > fa && r < fb)) r = 0.5 * (fa + fb);
  }
  return fb;
}

// One wavefront per particle: constants, support, partition edges (one per
// lane), work-item counts.
__global__ __launch_bounds__(64) void k_setup(Grid g, const double* __restrict__ params,
                                               int64_t n, const int32_t* __restrict__ np,
                                               int32_t np_uniform, int32_t stride, Tiling tl,
                                               const uint8_t* __restrict__ skip,
                                               PartConst* __restrict__ pc,
                                               int32_t* __restrict__ bounds,
                                               int32_t* __restrict__ cnt,
                                               int32_t* __restrict__ ptot,
                                               int32_t* __restrict__ widen) {
  const int lane = threadIdx.x & 63;
  const int64_t p = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (p >= n) return;                      // whole wavefronts
  const double* th = params + 6 * p;
  int npi = np ? np[p] : np_uniform;
  PartConst P;
  bool ok = true;
  for (int i = 0; i < 6; ++i) ok = ok && isfinite(th[i]);
  ok = ok && th[1] > 0.0 && fabs(th[2]) < 1.0 && th[5] >= 0.0 && npi >= 1 && npi <= stride;
  int32_t* bp = bounds + p * (int64_t)(stride + 1);
  int32_t* cp = cnt + p * (int64_t)stride;
  for (int l = lane; l < stride; l += 64) cp[l] = 0;
  if (lane == 0) ptot[p] = 0;
  P.np = npi;
  P.j_lo = 0; P.j_hi = -1;
  if (!ok) {
    P.status = kStatusInvalid;
    if (lane == 0) pc[p] = P;
    return;
  }
  if (skip && skip[p]) {  // outside the search box: not evaluated (let-them-fly)
    P.status = kStatusEmpty;
    if (lane == 0) pc[p] = P;
    return;
  }
  fill_constants(P, th);
  int last = (int)g.nbins - 1;
  double f_first = bin_freq(g, 0), f_last = bin_freq(g, last);
  const double t_end = tf_only(P, lane < 32 ? f_first : f_last);
  const double t_first = __shfl(t_end, 0, 64), t_last = __shfl(t_end, 32, 64);
  bool empty = (t_last < 0.0) || (t_first > g.T_obs);
  double flo = 0.0, fhi = 0.0;
  if (!empty) {
    const bool in_lo = t_first >= 0.0, in_hi = t_last <= g.T_obs;   // the band cuts the support
    if (!in_lo || !in_hi) {
      const bool need = lane < 32 ? !in_lo : !in_hi;
      const double root = invert_tf(P, lane < 32 ? 0.0 : g.T_obs, need, f_first, f_last, t_first,
                                    t_last, lane);
      flo = __shfl(root, 0, 64);
      fhi = __shfl(root, 32, 64);
    }
    if (in_lo) flo = f_first;
    if (in_hi) fhi = f_last;
    empty = !(flo <= fhi);
  }
  int jlo = 0, jhi = -1;
  if (!empty) {
    jlo = first_bin_at_or_above(g, flo, 0, last);
    // largest j with f_j <= fhi
    int j = first_bin_at_or_above(g, fhi, 0, last);
    if (j > last || bin_freq(g, j) > fhi) --j;
    jhi = j;
    empty = jlo > jhi;
  }
  P.flo = flo; P.fhi = fhi;
  if (empty) {
    P.status = kStatusEmpty;
    if (lane == 0) pc[p] = P;
    return;
  }
  P.status = kStatusOk;
  P.j_lo = jlo; P.j_hi = jhi;
  if (lane == 0) pc[p] = P;
  // edges e_l = flo + span l / Np: bin bp[l] is the first at or above e_l; each
  // lane computes both edges of its partitions (no exchange between lanes)
  const float mc53 = tl.mmax > 1 ? powf((float)P.mc_hi, 5.0f / 3.0f) : 0.f;
  const double span = fhi - flo;
  auto edge = [&](int l) -> int {
    if (l == 0) return jlo;
    if (l == npi) return jhi + 1;
    return first_bin_at_or_above(g, flo + (span * (double)l) / (double)npi, jlo, jhi);
  };
  int tot = 0;
  for (int l = lane; l < npi; l += 64) {
    const int a = edge(l), b = edge(l + 1);
    bp[l] = a;
    if (l == npi - 1) bp[npi] = b;
    int word = 1;
    if (tl.mmax > 1) widen[(int64_t)p * stride + l] = word = item_width(g, tl, mc53, a, b);
    ItemCut ic;
    const int c = item_count(tl, a, b, word, ic) * g.chan.n;
    cp[l] = c;
    tot += c;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) tot += __shfl_xor(tot, d, 64);
  if (lane == 0) ptot[p] = tot;
}

// Exclusive scan of cnt[m] into off[m] in three passes over blocks of
// kScanBlock counts: block sums, a one-block scan of the sums (which also
// writes *total and clears the exact-path counters), then each block's local
// scan plus its offset.
constexpr int kScanBlock = 4096;   // counts per block (1024 threads x 4)

template <typename T>
__device__ __forceinline__ T block_excl_scan(T x, T* sh, T& total) {
  // inclusive scan across the 1024 threads of the block (Hillis-Steele in LDS)
  const int t = threadIdx.x;
  sh[t] = x;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    T y = t >= o ? sh[t - o] : T(0);
    __syncthreads();
    sh[t] += y;
    __syncthreads();
  }
  total = sh[1023];
  T r = sh[t] - x;
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(1024) void k_scan_sums(const int32_t* __restrict__ cnt, int64_t m,
                                                    int32_t* __restrict__ bsum) {
  __shared__ int32_t red[1024];
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock + 4 * threadIdx.x;
  int32_t v = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) v += (i0 + e < m) ? cnt[i0 + e] : 0;
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

// nb <= 1024 * 4 block sums (m <= 16.7M counts), one block
__global__ __launch_bounds__(1024) void k_scan_top(int32_t* __restrict__ bsum, int32_t nb,
                                                   int32_t* __restrict__ total,
                                                   int32_t* __restrict__ ndirect,
                                                   int32_t* __restrict__ nrefine) {
  __shared__ int32_t sh[1024];
  const int i0 = 4 * threadIdx.x;
  int32_t v[4], x = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) { v[e] = (i0 + e < nb) ? bsum[i0 + e] : 0; x += v[e]; }
  int32_t tot;
  int32_t run = block_excl_scan(x, sh, tot);
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i0 + e < nb) { bsum[i0 + e] = run; run += v[e]; }
  if (threadIdx.x == 0) {
    total[0] = tot;
    ndirect[0] = 0;
    nrefine[0] = 0;
  }
}

__global__ __launch_bounds__(1024) void k_scan_apply(const int32_t* __restrict__ cnt, int64_t m,
                                                     const int32_t* __restrict__ bsum,
                                                     int32_t* __restrict__ off) {
  __shared__ int32_t sh[1024];
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock + 4 * threadIdx.x;
  int32_t v[4], x = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) { v[e] = (i0 + e < m) ? cnt[i0 + e] : 0; x += v[e]; }
  int32_t tot;
  int32_t run = block_excl_scan(x, sh, tot) + bsum[blockIdx.x];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i0 + e < m) { off[i0 + e] = run; run += v[e]; }
}

__global__ void k_fill(const int32_t* __restrict__ cnt, const int32_t* __restrict__ off, int64_t m,
                       const int32_t* __restrict__ bounds, const int32_t* __restrict__ widen,
                       int32_t stride, Tiling tl, int32_t nch, int2* __restrict__ items) {
  int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= m) return;
  int c = cnt[q], o = off[q];
  if (c == 0) return;
  const int64_t p = q / stride;
  const int32_t* bp = bounds + p * (stride + 1) + (q - p * stride);
  ItemCut ic;
  item_count(tl, bp[0], bp[1], tl.mmax > 1 ? widen[q] : 1, ic);
  for (int i = 0; i < c; ++i) items[o + i] = make_int2((int)q, item_word(i, ic, tl, nch));
}

// The same in one kernel for up to kScanOnce particles, one block each: a block
// sums the particles' totals before its own by itself (32 KB through L2 at
// most) instead of waiting for others, then scans its particle's counts and
// writes its work items; the last block writes the total.  all_exact: the exact
// loop takes every item.  Also clears the tile counters.  One launch instead of
// five: 4 us for one particle (17), 12 us at 4096 x 64 (31).
constexpr int64_t kScanOnce = 8192;

__global__ __launch_bounds__(256) void k_worklist(const int32_t* __restrict__ cnt,
                                                  const int32_t* __restrict__ bounds,
                                                  const int32_t* __restrict__ widen,
                                                  int32_t stride, Tiling tl, int32_t nch,
                                                  const int32_t* __restrict__ ptot,
                                                  int32_t* __restrict__ off,
                                                  int2* __restrict__ items,
                                                  int32_t* __restrict__ total,
                                                  int32_t* __restrict__ ndirect,
                                                  int32_t* __restrict__ nrefine, int all_exact,
                                                  int32_t* __restrict__ tcnt,
                                                  int32_t* __restrict__ tcur, int32_t n2,
                                                  int32_t* __restrict__ tile_ctr) {
  __shared__ int32_t s_off[257];
  __shared__ ItemCut s_cut[256];
  __shared__ int32_t s_wave[4];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int p = blockIdx.x;
  for (int i = p * 256 + t; i < n2; i += gridDim.x * 256) { tcnt[i] = 0; tcur[i] = 0; }
  if (p == 0 && t == 0) tile_ctr[0] = 0;
  int32_t before = 0;                              // items of the particles before this one
  for (int i = t; i < p; i += 256) before += ptot[i];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) before += __shfl_xor(before, d, 64);
  if (lane == 0) s_wave[wv] = before;
  __syncthreads();
  int32_t base = (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]);
  if (t == 0 && p == (int)gridDim.x - 1) {
    const int32_t tot = base + ptot[p];
    total[0] = tot;
    ndirect[0] = all_exact ? tot : 0;
    nrefine[0] = 0;
  }
  for (int l0 = 0; l0 < stride; l0 += 256) {
    const int l = l0 + t;
    const int64_t q = (int64_t)p * stride + l;
    const int32_t v = l < stride ? cnt[q] : 0;
    int32_t inc = v;                               // inclusive scan over the wavefront
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int32_t y = __shfl_up(inc, d, 64);
      if (lane >= d) inc += y;
    }
    __syncthreads();                               // s_wave, s_off of the part before
    if (lane == 63) s_wave[wv] = inc;
    __syncthreads();
    int32_t mine = 0, all = 0;
    for (int w = 0; w < 4; ++w) {
      if (w < wv) mine += s_wave[w];
      all += s_wave[w];
    }
    const int32_t o = mine + inc - v;
    s_off[t] = o;
    if (t == 0) s_off[256] = all;
    if (v > 0) {
      const int32_t* bp = bounds + (int64_t)p * (stride + 1) + l;
      item_count(tl, bp[0], bp[1], tl.mmax > 1 ? widen[q] : 1, s_cut[t]);
    }
    if (l < stride) off[q] = base + o;
    __syncthreads();
    for (int i = t; i < all; i += 256) {           // item -> its partition by bisection
      int lo = 0, hi = 256;                        // s_off[lo] <= i < s_off[hi]
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        const int mid = (lo + hi) >> 1;
        if (s_off[mid] <= i) lo = mid; else hi = mid;
      }
      items[base + i] = make_int2((int)((int64_t)p * stride + l0 + lo),
                                  item_word(i - s_off[lo], s_cut[lo], tl, nch));
    }
    base += all;
  }
}

// Prefix sums of the per-bin weight u (one channel): out[0] = 0,
// out[j + 1] = u_0 + ... + u_j.  The refinement estimate takes an item's
// sum of u from two entries.  Same three passes as the count scan.
__global__ __launch_bounds__(1024) void k_uscan_sums(const double* __restrict__ u, int64_t n,
                                                     double* __restrict__ bsum) {
  __shared__ double red[1024];
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock + 4 * threadIdx.x;
  double v = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) v += (i0 + e < n) ? u[i0 + e] : 0.0;
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(1024) void k_uscan_top(double* __restrict__ bsum, int32_t nb) {
  __shared__ double sh[1024];
  const int i0 = 4 * threadIdx.x;
  double v[4], x = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) { v[e] = (i0 + e < nb) ? bsum[i0 + e] : 0.0; x += v[e]; }
  double tot;
  double run = block_excl_scan(x, sh, tot);
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i0 + e < nb) { bsum[i0 + e] = run; run += v[e]; }
}

__global__ __launch_bounds__(1024) void k_uscan_apply(const double* __restrict__ u, int64_t n,
                                                      const double* __restrict__ bsum,
                                                      double* __restrict__ out) {
  __shared__ double sh[1024];
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock + 4 * threadIdx.x;
  double v[4], x = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) { v[e] = (i0 + e < n) ? u[i0 + e] : 0.0; x += v[e]; }
  double tot;
  double run = block_excl_scan(x, sh, tot) + bsum[blockIdx.x];
  if (blockIdx.x == 0 && threadIdx.x == 0) out[0] = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (i0 + e < n) { run += v[e]; out[i0 + e + 1] = run; }
}

// ---------------------------------------------------------------------------
// the hot loop, FP64
// ---------------------------------------------------------------------------
__device__ __forceinline__ void kahan_add(double& s, double& c, double x) {
  double y = x - c;
  double t = s + y;
  c = (t - s) - y;
  s = t;
}
__device__ __forceinline__ void kahan_addf(float& s, float& c, float x) {
  float y = x - c;
  float t = s + y;
  c = (t - s) - y;
  s = t;
}

// Sums of eight per-lane values over the wavefront in 10 exchanges instead of
// 8 x 6: each step hands half of the remaining values to the partner lane
// (xor 32, 16, 8), then the last value is summed over lanes xor 4, 2, 1.
// Returns the total of value number idx = 4 b5 + 2 b4 + b3 (b = lane bits);
// lanes with (lane & 7) == 0 hold the eight distinct totals.  Fixed order.
__device__ __forceinline__ double wave_sum8(const double* a, int lane, int& idx) {
  const bool h5 = (lane & 32) != 0, h4 = (lane & 16) != 0, h3 = (lane & 8) != 0;
  double b[4], c[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double keep = h5 ? a[4 + i] : a[i], give = h5 ? a[i] : a[4 + i];
    b[i] = keep + __shfl_xor(give, 32, 64);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = h4 ? b[2 + i] : b[i], give = h4 ? b[i] : b[2 + i];
    c[i] = keep + __shfl_xor(give, 16, 64);
  }
  double d = (h3 ? c[1] : c[0]) + __shfl_xor(h3 ? c[0] : c[1], 8, 64);
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
  idx = (h5 ? 4 : 0) + (h4 ? 2 : 0) + (h3 ? 1 : 0);
  return d;
}

// The same for four values: idx = 2 b5 + b4; lanes with (lane & 15) == 0
// hold the four totals.
__device__ __forceinline__ double wave_sum4(const double* a, int lane, int& idx) {
  const bool h5 = (lane & 32) != 0, h4 = (lane & 16) != 0;
  double b[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = h5 ? a[2 + i] : a[i], give = h5 ? a[i] : a[2 + i];
    b[i] = keep + __shfl_xor(give, 32, 64);
  }
  double d = (h4 ? b[1] : b[0]) + __shfl_xor(h4 ? b[0] : b[1], 16, 64);
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
  idx = (h5 ? 2 : 0) + (h4 ? 1 : 0);
  return d;
}

// (sin, cos)(2 pi k / kSinTab): copied to LDS by the kernels that read it per
// bin or node; the FP64 per-bin loop needs it only in the per-lane set-up of
// the difference recurrence and in the direct form (its LDS holds the tile)
__constant__ double2 c_sincos[kSinTab];
__constant__ double2 c_logtab[kLogTab];
// the same from the library's sincospi, for the exact loop (filled once per
// device; filling it in every block took 2 us of each launch)
__device__ double2 d_sincos[kSinTab];
__global__ void k_sincos_table() {
  const int k = threadIdx.x;
  double sv, cv;
  sincospi(2.0 * (double)k / (double)kSinTab, &sv, &cv);
  d_sincos[k] = make_double2(sv, cv);
}

constexpr int kSmallItem = 8;   // exact kernel: items this short share a wavefront
constexpr int kBigItem = 256;   // exact kernel: items longer than this take a whole block
constexpr int kSplitItem = 1024;   // ... and longer than this several, on very short lists
constexpr int kSplit = 4;
// where the blocks of a split item count themselves in its record: the unused
// integer beside the bin count (RecLayout::tail + 4), zero from the node kernel
template <bool MIXED> struct RecSplit { static constexpr int count = MIXED ? 85 : 109; };   // int index

// Exact per-bin template loop.  FP64 (MIXED = false): everything in FP64,
// Kahan-compensated per-lane sums.  Mixed (MIXED = true): the phase, the orbit
// and the TDI response are evaluated in FP64 exactly as on the FP64 path and
// rounded once to FP32; the products with the FP32 data and the N-term sums
// (Z+, Zx) are FP32 with Kahan compensation, the M-terms (P, Q, R) are FP64
// sums of the rounded response.  The response is not computed in FP32: its
// sinc factors are formed from sin(x0 (1 +- k.n)) by angle addition and the
// two arms' contributions are subtracted, and in FP32 both cancel (relative
// errors of 1e-6..1e-5 for sources near an arm direction), which tilts the
// (T+, Tx) direction; the statistic amplifies such a tilt by ~sqrt(cond M) in
// the weak eigen-direction of the short, ill-conditioned partitions this
// kernel serves.  Rounding a correct response to FP32 tilts it by ~6e-8 only.
template <bool MIXED>
__global__ __launch_bounds__(256, 3) void k_eval_exact(Grid g,
                                                    const PartConst* __restrict__ pc,
                                                    const int32_t* __restrict__ bounds, int32_t stride,
                                                    const int2* __restrict__ items,
                                                    const int32_t* __restrict__ total, Tiling tl,
                                                    const double* __restrict__ wr,
                                                    const double* __restrict__ wi,
                                                    const double* __restrict__ u,
                                                    const float* __restrict__ wr32,
                                                    const float* __restrict__ wi32,
                                                    const float* __restrict__ u32,
                                                    const double* __restrict__ s0a,
                                                    const double* __restrict__ c0a,
                                                    const double* __restrict__ ek,
                                                    double* __restrict__ rec,
                                                    double* __restrict__ partials,
                                                    const int32_t* __restrict__ sel,
                                                    const int32_t* __restrict__ nsel) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int nwaves = (gridDim.x * blockDim.x) >> 6;
  const int W = sel ? nsel[0] : total[0];
  if (W == 0) return;
  __shared__ double2 s_tab[kSinTab];              // coarse angles of the template's sin/cos
  __shared__ double s_red[4][8];                  // per-wave sums of a block-wide item
  for (int i = threadIdx.x; i < kSinTab; i += blockDim.x) s_tab[i] = d_sincos[i];
  __syncthreads();
  // The eight partition terms of bin j for the item (q, c) of a particle;
  // on the mixed path t[0..3] are FP32 products (widened).
  auto terms = [&](int q, int c, int j, double t[8]) {
    const int p = q / stride;
    const PartConst& P = pc[p];
    const int ch = item_chan(c, tl, g.chan.n);
    const int64_t co = (int64_t)ch * g.nbins;   // the channel's data
    const double* ekq = (ek && P.sur) ? ek + 8 * (int64_t)q : nullptr;
    double f = bin_freq(g, j);
    double cps, sps, tpr, tpi, txr, txi;
    template_fp64(P, f, s0a[j], c0a[j], cps, sps, tpr, tpi, txr, txi, ekq, g.chan.code[ch],
                  &g.orb, s_tab);
    if constexpr (MIXED) {
      const float cf = (float)cps, sf = (float)sps;
      const float pr = (float)tpr, pi = (float)tpi, xr = (float)txr, xi = (float)txi;
      const float a = wr32[co + j], b = wi32[co + j];
      const float Wr = a * cf - b * sf, Wi = a * sf + b * cf;   // w e^{i Phi}
      t[0] = (double)(Wr * pr + Wi * pi);
      t[1] = (double)(Wi * pr - Wr * pi);
      t[2] = (double)(Wr * xr + Wi * xi);
      t[3] = (double)(Wi * xr - Wr * xi);
      tpr = pr; tpi = pi; txr = xr; txi = xi;     // M-terms from the same rounded response
      const double uu = (double)u32[co + j];
      t[4] = uu * (tpr * tpr + tpi * tpi);
      t[5] = uu * (txr * txr + txi * txi);
      t[6] = uu * (tpr * txr + tpi * txi);
      t[7] = uu * (tpi * txr - tpr * txi);
    } else {
      double a = wr[co + j], b = wi[co + j], uu = u[co + j];
      double Wr = a * cps - b * sps, Wi = a * sps + b * cps;   // w e^{i Phi}
      t[0] = Wr * tpr + Wi * tpi;     // Z+ = sum W conj(T'+)
      t[1] = Wi * tpr - Wr * tpi;
      t[2] = Wr * txr + Wi * txi;     // Zx
      t[3] = Wi * txr - Wr * txi;
      t[4] = uu * (tpr * tpr + tpi * tpi);
      t[5] = uu * (txr * txr + txi * txi);
      t[6] = uu * (tpr * txr + tpi * txi);   // R = sum u T'+ conj(T'x)
      t[7] = uu * (tpi * txr - tpr * txi);
    }
  };
  auto bins_of = [&](int w, int& q, int& c, int& b0, int& b1) {
    const int2 it = items[w];
    q = it.x;
    c = it.y;
    const int p = q / stride, l = q - p * stride;
    const int32_t* bp = bounds + (int64_t)p * (stride + 1);
    item_bins(bp[l], bp[l + 1], c, item_chan(c, tl, g.chan.n), tl, b0, b1);
  };
  // All items, or only those listed in sel (the interpolating kernel's
  // rejects and refinements).  Items of at most kSmallItem bins go 32 list
  // entries to a wavefront, two, four or eight lanes each (the fewest that hold
  // the longest of them: 32, 16 or 8 at a time; one bin per lane, then a fixed
  // butterfly, whose result does not depend on the width); larger ones one per
  // wavefront in a second sweep over the list, so that a list of long items
  // (the refinement pass) spreads over the whole grid, and on a short list
  // those above kBigItem bins one per block (or four) in a third.  Each sweep's
  // lanes load the items' bounds for many entries at a time (one entry at a
  // time, the chain of dependent loads set the pass's length on the 24,910 items of
  // a small swarm: 27 us).  Which path an item takes depends
  // on the item and the list's length alone, so its sums do not depend on the
  // order of the list.
  const int G = (W + 31) >> 5;
  for (int gi = wave; gi < G; gi += nwaves) {
    const int slot = gi * 32 + (lane & 31);
    int w = 0, q = 0, c = 0, b0 = 0, b1 = 0;
    if (slot < W) {
      w = sel ? sel[slot] : slot;
      bins_of(w, q, c, b0, b1);
    }
    const int nb = b1 - b0 <= kSmallItem ? b1 - b0 : 0;      // 0: not of this sweep
    if (!__any(nb > 0)) continue;
    const int width = __any(nb > 4) ? 8 : (__any(nb > 2) ? 4 : 2), at = 64 / width;
    for (int i0 = 0; i0 < 32; i0 += at) {
      const int src = i0 + lane / width, e = lane & (width - 1);
      const int wi = __shfl(w, src, 64), qi = __shfl(q, src, 64), ci = __shfl(c, src, 64);
      const int j = __shfl(b0, src, 64) + e, ni = __shfl(nb, src, 64);
      double t[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) t[i] = 0.0;
      if (e < ni) terms(qi, ci, j, t);
      for (int d = width >> 1; d > 0; d >>= 1)
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] += __shfl_xor(t[i], d, 64);
      if (ni > 0 && e == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) partials[(int64_t)wi * 8 + i] = t[i];
      }
    }
  }
  // Kahan-compensated sums of this thread's bins j0, j0 + step, ... < j1 of
  // one item (true sum ~ acc - cmp, returned compensated): the partition
  // matrix can have cond ~ 1e5..1e8, which amplifies summation error.
  auto thread_sums = [&](int qb, int cb, int j0, int j1, int step, double* acc) {
    double cmp[8];
    float accf[4], cmpf[4];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = cmp[i] = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) accf[i] = cmpf[i] = 0.0f;
    for (int j = j0; j < j1; j += step) {
      double tt[8];
      terms(qb, cb, j, tt);
      if constexpr (MIXED) {
#pragma unroll
        for (int i = 0; i < 4; ++i) kahan_addf(accf[i], cmpf[i], (float)tt[i]);
#pragma unroll
        for (int i = 4; i < 8; ++i) kahan_add(acc[i], cmp[i], tt[i]);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) kahan_add(acc[i], cmp[i], tt[i]);
      }
    }
    if constexpr (MIXED) {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = (double)accf[i] - (double)cmpf[i];
#pragma unroll
      for (int i = 4; i < 8; ++i) acc[i] -= cmp[i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] -= cmp[i];
    }
  };
  // A short list (rejects, refinement) leaves most wavefronts idle while a few
  // take its long items: there items above kBigItem bins take a whole block.
  // A long list (every item, FSTAT_EVAL_EXACT) fills the grid one item per
  // wavefront.
  const bool by_block = W < 4 * nwaves;
  // items of kSmallItem + 1 bins and more (up to kBigItem for a short list):
  // one per wavefront
  for (int s0 = wave; s0 < W; s0 += 64 * nwaves) {
    const int slot = s0 + lane * nwaves;
    int w = 0, q = 0, c = 0, b0 = 0, b1 = 0;
    if (slot < W) {
      w = sel ? sel[slot] : slot;
      bins_of(w, q, c, b0, b1);
    }
    const int nb = b1 - b0;
    for (uint64_t todo = __ballot(nb > kSmallItem && !(by_block && nb > kBigItem)); todo != 0;
         todo &= todo - 1) {
      const int l = __builtin_ctzll(todo);       // the same on every lane: scalar indices
      const int wb = __builtin_amdgcn_readlane(w, l), qb = __builtin_amdgcn_readlane(q, l);
      const int cb = __builtin_amdgcn_readlane(c, l);
      const int bb0 = __builtin_amdgcn_readlane(b0, l), bb1 = __builtin_amdgcn_readlane(b1, l);
      double acc[8];
      thread_sums(qb, cb, bb0 + lane, bb1, 64, acc);
      int idx;
      const double tot = wave_sum8(acc, lane, idx);
      if ((lane & 7) == 0) partials[(int64_t)wb * 8 + idx] = tot;
    }
  }
  if (!by_block) return;
  // longer items: one per block (a few long rejects or refined items would
  // otherwise each hold one wavefront for the whole pass); the four waves'
  // sums are added in a fixed order.  On a list of at most a quarter of the
  // blocks, items above kSplitItem bins take four blocks, whose sums meet in the
  // item's record (its interpolants are not needed any more) and are added in
  // order by the last of them (5120 bins by one block: ~50 us of latency for a
  // single template).
  const int parts = sel && (int64_t)W * kSplit <= (int64_t)gridDim.x ? kSplit : 1;
  for (int64_t u0 = blockIdx.x; u0 < (int64_t)W * parts; u0 += 64 * (int64_t)gridDim.x) {
    const int64_t u = u0 + (int64_t)lane * gridDim.x;
    const int slot = (int)(u / parts), part = (int)(u - (int64_t)slot * parts);
    int w = 0, q = 0, c = 0, b0 = 0, b1 = 0;
    if (slot < W) {
      w = sel ? sel[slot] : slot;
      bins_of(w, q, c, b0, b1);
    }
    const int nb = b1 - b0;
    // the same on every wave of the block
    for (uint64_t todo = __ballot(nb > kBigItem && (part == 0 || nb > kSplitItem)); todo != 0;
         todo &= todo - 1) {
      const int l = __builtin_ctzll(todo);
      const int wb = __builtin_amdgcn_readlane(w, l), qb = __builtin_amdgcn_readlane(q, l);
      const int cb = __builtin_amdgcn_readlane(c, l), pb = __builtin_amdgcn_readlane(part, l);
      int bb0 = __builtin_amdgcn_readlane(b0, l), bb1 = __builtin_amdgcn_readlane(b1, l);
      const bool split = parts > 1 && bb1 - bb0 > kSplitItem;
      if (split) {
        const int n = (bb1 - bb0 + kSplit - 1) / kSplit;
        bb0 += pb * n;
        bb1 = min(bb1, bb0 + n);
      }
      double acc[8];
      thread_sums(qb, cb, bb0 + (int)threadIdx.x, bb1, (int)blockDim.x, acc);
      int idx;
      const double tot = wave_sum8(acc, lane, idx);
      if ((lane & 7) == 0) s_red[threadIdx.x >> 6][idx] = tot;
      __syncthreads();
      double sum = 0.0;
      if (threadIdx.x < 8)
        sum = ((s_red[0][threadIdx.x] + s_red[1][threadIdx.x]) + s_red[2][threadIdx.x]) +
              s_red[3][threadIdx.x];
      if (!split) {
        if (threadIdx.x < 8) partials[(int64_t)wb * 8 + threadIdx.x] = sum;
      } else if (threadIdx.x < 64) {             // one wavefront: its stores, then its count
        double* r = rec + (int64_t)wb * kInterpRec;
        int* arrived = reinterpret_cast<int*>(r) + RecSplit<MIXED>::count;
        if (threadIdx.x < 8)
          __hip_atomic_store(r + 8 * pb + threadIdx.x, sum, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();
        int old = 0;
        if (threadIdx.x == 0)
          old = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        old = __builtin_amdgcn_readfirstlane(old);
        if (old == kSplit - 1) {
          __threadfence();
          if (threadIdx.x < 8) {
            double x = 0.0;
            for (int k = 0; k < kSplit; ++k)
              x += __hip_atomic_load(r + 8 * k + threadIdx.x, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
            partials[(int64_t)wb * 8 + threadIdx.x] = x;
          }
          if (threadIdx.x == 0)
            __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      __syncthreads();                           // s_red is rewritten by the next item
    }
  }
}

// ---------------------------------------------------------------------------
// the hot loop, interpolating form (default)
// ---------------------------------------------------------------------------
// Within one work item (at most a tile of consecutive bins of one partition)
// every factor of the template except the fast phase is smooth in f, and the
// phase is smooth once a linear term is taken out.  Per item, with m = j - b0
// and s = 2 m / (nb - 1) - 1 in [-1, 1]:
//   Phi(m) / (2 pi) = Phi_0 + B m + R(s),   R(-1) = R(+1) = 0 up to rounding,
// where Phi_0 is the whole phase (cycles, double-double) at the first bin and
// B the secant slope to the last bin; R and the four real components of the
// transfer (T''_+, T''_x) are replaced by their degree-9 interpolants through
// the 10 Chebyshev points of the first kind, written as monomials in s.  The
// node values and the two end-point values are evaluated exactly
// (template_node); an item whose interpolants miss either end point by more
// than 1e-12 cycles (phase; the exact phase itself carries ~1e-13) or 2e-13 of
// the largest transfer component, or that has fewer than kMinInterp bins,
// goes to the exact per-bin kernels (sel list).
// Items whose interpolation error could move their partition's F by more
// than the plan's refinement budget (default 5e-10, relative; the first-order
// estimate of k_mark) are evaluated again exactly.
// Node evaluation packs 5 items x 12 points onto one wavefront's lanes.
constexpr int kCheb = 10;
constexpr int kLanesItem = kCheb + 2;
constexpr int kItemsWave = 5;
constexpr int kMinInterp = 32;
constexpr double kInterpTolPhase = 1e-12;
constexpr double kInterpTolT = 2e-13;
constexpr int kUnitItems = 64;      // items per scheduling unit of the bin loop
constexpr double kTruncFloor = 6e-14;  // FP64 transfer truncation allowance
// Difference recurrence of the FP64 bin loop: shortest lane run that takes
// it (below, the set-up of about 160 operations per lane costs more than the
// ~15 it saves per bin), the largest |phi| of its series, and the largest
// phase error allowed from the neglected fifth difference [rad].
constexpr int kRecMinRun = 9;
constexpr double kRecPhiMax = 4e-3;
constexpr double kRecTrunc = 1e-13;
constexpr double kTwoPi = 6.283185307179586477;
// kStirF[k][j] = j! S(k, j) (S: Stirling numbers of the second kind), the
// j-th forward difference of t^k at t = 0; equivalently
// t^k = sum_j kStirF[k][j] C(t, j)
constexpr double kStirF[kCheb][kCheb] = {
    {1, 0, 0, 0, 0, 0, 0, 0, 0, 0},
    {0, 1, 0, 0, 0, 0, 0, 0, 0, 0},
    {0, 1, 2, 0, 0, 0, 0, 0, 0, 0},
    {0, 1, 6, 6, 0, 0, 0, 0, 0, 0},
    {0, 1, 14, 36, 24, 0, 0, 0, 0, 0},
    {0, 1, 30, 150, 240, 120, 0, 0, 0, 0},
    {0, 1, 62, 540, 1560, 1800, 720, 0, 0, 0},
    {0, 1, 126, 1806, 8400, 16800, 15120, 5040, 0, 0},
    {0, 1, 254, 5796, 40824, 126000, 191520, 141120, 40320, 0},
    {0, 1, 510, 18150, 186480, 834120, 1905120, 2328480, 1451520, 362880}};

__constant__ double c_cheb_s[kCheb];          // nodes cos(pi (k + 1/2) / 10)
// Row tables of the node kernel, indexed [node kn][lane k of the item]: on a
// node lane (k < kCheb) the map node value kn -> monomial coefficient of s^k
// of the interpolant, on the end lanes k = kCheb, kCheb + 1 the map node
// value kn -> interpolant at s = -1, +1.
__constant__ double c_row9[kCheb][kLanesItem];      // degree-9 interpolant
// The mixed path's transfer interpolants: the Chebyshev series truncated
// after degree kDegT (its error, ~1e-10 on paper-scale items, is far below FP32
// rounding); node rows above kDegT are zero.  Items whose series truncated
// after degree kDegTLow stays within kInterpTolTMixed at both ends take that
// one (4 FP32 additions per bin fewer); degree 4 for every item would
// send enough items to the exact loop to cost more than it saves.
constexpr int kDegT = 6;
constexpr int kDegTLow = 4;
__constant__ double c_row6[kCheb][kLanesItem];
__constant__ double c_row4[kCheb][kLanesItem];
// Mixed loop: forward differences of the phase carried per bin where the
// rest may be dropped, and the largest phase error [turns] that dropping them
// may cause (the FP32 sine's own error is ~1e-7 turns).
constexpr int kMixDiff = 4;
constexpr double kMixTrunc = 1e-9;
// The FP64 loop's transfer interpolants may be truncated after degree 5 or 7
// per item when that keeps them within the item's own error (most paper-scale
// items need 5-7 of the 10 Chebyshev terms at the 2e-13 bar).
__constant__ double c_rowt[2][kCheb][kLanesItem];   // [0]: degree 5, [1]: degree 7
// Quadrature of an item's interpolant: sum over its bins of the degree-9
// interpolant through the nodes = sum_k W_k g(s_k), W_k = sum_j c_jk S_j(nb)
// with c_jk the node-to-Chebyshev-coefficient map and S_j(nb) = sum_m T_j(s_m)
// (zero for odd j: the bins are symmetric in s).  c_cheb_D[i][k] = c_{2i,k}.
__constant__ double c_cheb_D[5][kCheb];
// Least-squares fit of u on a u-tile: inverse Gram matrix of T_0..T_9 on the
// kUTile equispaced points s_m = 2m/(kUTile-1) - 1.
__constant__ double c_ufit_Ginv[kUCoef][kUCoef];

__device__ __forceinline__ double readlane_d(double x, int l) {
  int2 v = *reinterpret_cast<int2*>(&x);
  v.x = __builtin_amdgcn_readlane(v.x, l);
  v.y = __builtin_amdgcn_readlane(v.y, l);
  return *reinterpret_cast<double*>(&v);
}

template <typename T>
__device__ __forceinline__ T horner(const T* c, T s) {
  T r = c[kCheb - 1];
#pragma unroll
  for (int n = kCheb - 2; n >= 0; --n) r = r * s + c[n];
  return r;
}

template <int D, typename T>
__device__ __forceinline__ T horner_n(const T* c, T s) {
  T r = c[D];
#pragma unroll
  for (int n = D - 1; n >= 0; --n) r = r * s + c[n];
  return r;
}

// The same degree-9 polynomial by Estrin's scheme, with the powers s^2, s^4,
// s^8 shared by the five polynomials of a bin: 9 FMAs as in Horner's rule,
// but a dependency depth of 4 instead of 9.
static_assert(kCheb == 10, "estrin9 is written for degree 9");
__device__ __forceinline__ double estrin9(const double* c, double s, double s2, double s4,
                                          double s8) {
  const double q01 = fma(c[1], s, c[0]), q23 = fma(c[3], s, c[2]);
  const double q45 = fma(c[5], s, c[4]), q67 = fma(c[7], s, c[6]);
  const double q89 = fma(c[9], s, c[8]);
  const double a = fma(q23, s2, q01), b = fma(q67, s2, q45);
  return fma(q89, s8, fma(b, s4, a));
}

// Degree-D Estrin forms of the same monomial series (D = 5, 7) for the FP64
// loop's transfer interpolants truncated by the node kernel.
template <int D>
__device__ __forceinline__ double estrin_d(const double* c, double s, double s2, double s4,
                                           double s8) {
  static_assert(D == 5 || D == 7 || D == 9, "degree 5, 7 or 9");
  if constexpr (D == 9) {
    return estrin9(c, s, s2, s4, s8);
  } else if constexpr (D == 7) {
    const double q01 = fma(c[1], s, c[0]), q23 = fma(c[3], s, c[2]);
    const double q45 = fma(c[5], s, c[4]), q67 = fma(c[7], s, c[6]);
    return fma(fma(q67, s2, q45), s4, fma(q23, s2, q01));
  } else {
    const double q01 = fma(c[1], s, c[0]), q23 = fma(c[3], s, c[2]);
    const double q45 = fma(c[5], s, c[4]);
    return fma(q45, s4, fma(q23, s2, q01));
  }
}

// Per-item interpolation record: monomial coefficients of R (kCheb), then of
// Re T''_+, Im T''_+, Re T''_x, Im T''_x (nT each: kCheb, or kDegT + 1 on the
// mixed path), then A = frac(Phi_0), B' = B - rint(B), B, two integers (the
// item's flags and its first bin), two more (its bin count; unused), the step
// alpha = 2 / (bins - 1) of s per bin and -B / df (so that the bin loops need
// nothing else per item, and no division).  Flags: the loop that takes the
// item (kRecExact .. kRecBlocks), the degree its transfer interpolants are
// evaluated at << 8, its channel << 16.
constexpr int kRec = 5 * kCheb + 7;
static_assert(kRec == kInterpRec && kRec <= 64, "record layout");
template <bool MIXED> struct RecLayout {
  static constexpr int nT = MIXED ? kDegT + 1 : kCheb;
  static constexpr int tail = kCheb + 4 * nT;   // A, B', B, {flags, b0}, {bins, -}, alpha, -B/df
};
// the split items of the exact loop count their blocks in the record's unused
// integer (half 1 of tail + 4) and keep kSplit sets of eight sums below it
template <bool MIXED> struct RecSplitCheck {
  static_assert(2 * (RecLayout<MIXED>::tail + 4) + 1 == RecSplit<MIXED>::count, "record layout");
  static_assert(8 * kSplit <= RecLayout<MIXED>::tail, "room for the sums");
};
template struct RecSplitCheck<false>;
template struct RecSplitCheck<true>;
// the per-bin loop marks the items whose lanes took its short form (the
// difference recurrence; mixed: four phase differences) for fstat_interp_stats
enum { kRecExact = 0, kRecBins = 1, kRecBinsShort = 2, kRecBlocks = 3 };
__device__ __forceinline__ int rec_int(const double& x, int half) {
  return reinterpret_cast<const int*>(&x)[half];
}

// Chebyshev series sum_k c_k T_k(x) (Clenshaw).
__device__ __forceinline__ double cheb_eval10(const double* __restrict__ c, double x) {
  double b1 = 0.0, b2 = 0.0;
  const double x2 = 2.0 * x;
#pragma unroll
  for (int k = kUCoef - 1; k >= 1; --k) {
    const double b0 = fma(x2, b1, c[k] - b2);
    b2 = b1;
    b1 = b0;
  }
  return fma(x, b1, c[0] - b2);
}

// S_j(nb) = sum_{m < nb} T_j(2m/(nb-1) - 1) for j = 0, 2, .., 8, one nb per
// thread (Neumaier sums); S_j(1) = T_j(0) stands for the single bin at s = 0
// and S_j(0) = 0.
__global__ void k_cheb_sums(double* __restrict__ out) {
  const int nb = blockIdx.x * blockDim.x + threadIdx.x;
  if (nb > kSsumMax) return;
  double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, e[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int m = 0; m < nb; ++m) {
    const double s = nb > 1 ? 2.0 * (double)m / (double)(nb - 1) - 1.0 : 0.0;
    double tv[9];
    tv[0] = 1.0;
    tv[1] = s;
#pragma unroll
    for (int j = 2; j <= 8; ++j) tv[j] = fma(2.0 * s, tv[j - 1], -tv[j - 2]);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const double x = tv[2 * i], tt = a[i] + x;
      e[i] += (fabs(a[i]) >= fabs(x)) ? (a[i] - tt) + x : (x - tt) + a[i];
      a[i] = tt;
    }
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) out[i * (kSsumMax + 1) + nb] = a[i] + e[i];
}

// Fit of u on each u-tile (one block of kUTile threads per tile): Chebyshev
// coefficients by least squares and the largest residual relative to the
// tile's largest |u|; a partial last tile is left unfit (residual inf).
__global__ __launch_bounds__(kUTile) void k_ufit(const double* __restrict__ u, int64_t nbins,
                                                 int32_t ntiles, double* __restrict__ coef,
                                                 double* __restrict__ resid) {
  __shared__ double red[kUCoef][kUTile / 64];
  __shared__ double c_s[kUCoef];
  __shared__ double mx[2][kUTile / 64];
  const int tile = blockIdx.x;
  const int m = threadIdx.x, lane = m & 63, wv = m >> 6;
  if (tile >= ntiles) return;
  const int64_t j = (int64_t)tile * kUTile + m;
  const bool full = (int64_t)(tile + 1) * kUTile <= nbins;
  const double um = (j < nbins) ? u[j] : 0.0;
  const double s = 2.0 * (double)m / (double)(kUTile - 1) - 1.0;
  double tk[kUCoef];
  tk[0] = 1.0;
  tk[1] = s;
#pragma unroll
  for (int k = 2; k < kUCoef; ++k) tk[k] = fma(2.0 * s, tk[k - 1], -tk[k - 2]);
#pragma unroll
  for (int k = 0; k < kUCoef; ++k) {
    double v = um * tk[k];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) red[k][wv] = v;
  }
  __syncthreads();
  if (m < kUCoef) {
    double c = 0.0;
#pragma unroll
    for (int k = 0; k < kUCoef; ++k) {
      double b = 0.0;
#pragma unroll
      for (int w = 0; w < kUTile / 64; ++w) b += red[k][w];
      c = fma(c_ufit_Ginv[m][k], b, c);
    }
    c_s[m] = c;
    if (full) coef[(int64_t)tile * kUCoef + m] = c;
    else coef[(int64_t)tile * kUCoef + m] = 0.0;
  }
  __syncthreads();
  double r = (j < nbins) ? fabs(um - cheb_eval10(c_s, s)) : 0.0, a = fabs(um);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    r = fmax(r, __shfl_xor(r, o, 64));
    a = fmax(a, __shfl_xor(a, o, 64));
  }
  if (lane == 0) { mx[0][wv] = r; mx[1][wv] = a; }
  __syncthreads();
  if (m == 0) {
    double rr = 0.0, aa = 0.0;
    for (int w = 0; w < kUTile / 64; ++w) { rr = fmax(rr, mx[0][w]); aa = fmax(aa, mx[1][w]); }
    resid[tile] = !full ? __builtin_inf() : (aa > 0.0 ? rr / aa : 0.0);
  }
}
// tolerances of the end-point check on the mixed path (FP32 products; its
// node phases are plain FP64, ~2e-9 cycles of rounding at 1e7 cycles, which
// the interpolant carries to its end points a few times over; the FP32 sine
// resolves ~6e-8 turns)
constexpr double kInterpTolPhaseMixed = 1e-7;
constexpr double kInterpTolTMixed = 3e-8;

// Node values, coefficients and end-point check of every work item (all
// lanes active: lanes 60..63 repeat the last point of the last item).  TAB:
// the plan has a numerical orbit (a separate instance keeps the table code
// out of the analytic kernel's registers).
//
// Bound by FP64 issue (~1,600 vector operations per five items, 456 B written per
// item) and, below that, by how many waves cover its dependent chains: what kept
// it at two waves per SIMD was values held across the per-particle loop and the
// library's sine and logarithm, so the loop hands its results over in LDS and
// sine, logarithm and x^{-1/9} come from tables and a third-order step; three
// waves with numerical orbits' tables would spill (orbit batch 1.29 -> 1.48 ms).
// 1.67 M items FP64: 1.71 -> 1.30 ms; 0.97 M mixed: 0.85 -> 0.59 ms.
//
// With block spectra (sp.L > 0) an item goes to the block loop when over any
// of its blocks the phase stays within sp.psi radians of a straight line and
// its slope within half a slot of the spectra's range, and it ends below the
// spectra's fmax; otherwise to the per-bin loop.  sup |R'| and sup |R''| are
// bounded by the coefficients' sums.
struct SpecShape {
  int32_t L, Q, nslots, nblk;
  double psi;
  double hq, smax;      // half a slot of the slope grid, its last slot
  double fmax;          // see Spectra
};
template <bool MIXED, bool TAB>
__global__ __launch_bounds__(256, TAB ? 2 : 3) void k_interp_nodes(Grid g,
                                                      const PartConst* __restrict__ pc,
                                                      const int32_t* __restrict__ bounds,
                                                      int32_t stride,
                                                      const int2* __restrict__ items,
                                                      const int32_t* __restrict__ total,
                                                      Tiling tl,
                                                      const double* __restrict__ ek,
                                                      double* __restrict__ rec,
                                                      uint8_t* __restrict__ xflag,
                                                      float2* __restrict__ xerr,
                                                      int32_t* __restrict__ direct,
                                                      int32_t* __restrict__ ndirect,
                                                      UModel um,
                                                      double* __restrict__ partials,
                                                      SpecShape sp, double rstride) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int nwaves = (gridDim.x * blockDim.x) >> 6;
  const int W = total[0];
  const int G = (W + kItemsWave - 1) / kItemsWave;
  if (blockIdx.x * (blockDim.x >> 6) >= G) return;   // more blocks than groups of items
  __shared__ double2 s_tab[kSinTab];              // coarse angles of the template's sin/cos
  // the row tables in LDS (the coefficient loop reads one entry of each per
  // node and lane; from the constant tables each read is a vector memory load)
  __shared__ double s_r9[kCheb][kLanesItem], s_rT[kCheb][kLanesItem];
  __shared__ double s_rt[MIXED ? 1 : 2][kCheb][kLanesItem];
  // each lane's node values, read back by the lanes of its item (one write,
  // broadcast reads: LDS operations of one wave complete in order)
  constexpr int kNd = 14;
  __shared__ __align__(16) double s_nd[4][64][kNd];
  double* my_nd = s_nd[threadIdx.x >> 6][lane];
  for (int i = threadIdx.x; i < kCheb * kLanesItem; i += blockDim.x) {
    const int kn = i / kLanesItem, kk = i - kn * kLanesItem;
    s_r9[kn][kk] = c_row9[kn][kk];
    s_rT[kn][kk] = MIXED ? c_row6[kn][kk] : c_row9[kn][kk];
    if constexpr (!MIXED) {
      s_rt[0][kn][kk] = c_rowt[0][kn][kk];
      s_rt[1][kn][kk] = c_rowt[1][kn][kk];
    } else {
      s_rt[0][kn][kk] = c_row4[kn][kk];
    }
  }
  __shared__ double2 s_log[kLogTab];
  for (int i = threadIdx.x; i < kSinTab; i += blockDim.x) s_tab[i] = c_sincos[i];
  for (int i = threadIdx.x; i < kLogTab; i += blockDim.x) s_log[i] = c_logtab[i];
  __syncthreads();
  const int q = min(lane / kLanesItem, kItemsWave - 1);
  const int k = min(lane - q * kLanesItem, kLanesItem - 1);
  const int base = q * kLanesItem;
  // a group's items are loaded two groups ahead and its bounds one ahead
  auto load_item = [&](int grp) { return items[min(min(grp, G - 1) * kItemsWave + q, W - 1)]; };
  auto bounds_of = [&](int2 it, int& p) {
    p = div_by(it.x, rstride);
    const int32_t* bp = bounds + (int64_t)p * (stride + 1) + (it.x - p * stride);
    return make_int2(bp[0], bp[1]);
  };
  if (wave >= G) return;
  int2 it1 = load_item(wave), it2 = load_item(wave + nwaves);
  int p1;
  int2 bd1 = bounds_of(it1, p1);
  for (int grp = wave; grp < G; grp += nwaves) {
    const int w = min(grp * kItemsWave + q, W - 1);
    const int2 it = it1, bd = bd1;
    const int p = p1;
    it1 = it2;
    it2 = load_item(grp + 2 * nwaves);
    bd1 = bounds_of(it1, p1);
    const int ch = item_chan(it.y, tl, g.chan.n);
    int b0, b1;
    item_bins(bd.x, bd.y, it.y, ch, tl, b0, b1);
    const int nb = b1 - b0;
    if (!__any(nb >= kMinInterp)) {
      // no item of this group is long enough to interpolate: all of them go
      // to the exact loop without evaluating their nodes
      if (k == kCheb && lane - base < kLanesItem && grp * kItemsWave + q < W) {
        xflag[w] = kItemExact;
        direct[atomicAdd(ndirect, 1)] = w;
      }
      continue;
    }
    const double sk = k < kCheb ? c_cheb_s[k] : (k == kCheb ? -1.0 : 1.0);
    const double mk = (sk + 1.0) * 0.5 * (double)(nb > 1 ? nb - 1 : 0);
    // exact frequency (k_lo + b0 + mk) df of the node, as double-double
    const dd f = dd_add(two_prod((double)(g.k_lo + b0), g.df), two_prod(mk, g.df));
    // (their results go through the lane's slots: carried in registers, the
    // earlier turns' values would be live beside those being formed)
    // the lanes of one particle at a time (nearly always all of them): its
    // constants come through the scalar cache into scalar registers
    for (uint64_t todo = __ballot(true); todo != 0;) {
      const int pu = __builtin_amdgcn_readlane(p, __builtin_ctzll(todo));
      int ps = pu;
      asm("" : "+s"(ps));   // not p itself: the compiler would put it back where they are equal
      const kconst_PartConst* kp = (const kconst_PartConst*)(uintptr_t)(pc + ps);
      todo &= ~__ballot(p == pu);
      if (p == pu) {
        const PartConst P = load_particle(kp);
        const double* ekq = (ek && P.sur) ? ek + 8 * (int64_t)it.x : nullptr;
        double t1, t2, t3, t4;
        dd ph;
        if constexpr (MIXED)
          ph = dd{template_node_fp64(P, f.hi, ekq, t1, t2, t3, t4, g.chan.code[ch],
                                     TAB ? &g.orb : nullptr, s_tab, s_log), 0.0};
        else
          ph = template_node(P, f, ekq, t1, t2, t3, t4, g.chan.code[ch],
                             TAB ? &g.orb : nullptr, s_tab, s_log);
        my_nd[0] = ph.hi; my_nd[1] = ph.lo;
        my_nd[2] = t1; my_nd[3] = t2; my_nd[4] = t3; my_nd[5] = t4;
      }
    }
    __builtin_amdgcn_wave_barrier();
    const dd ph{my_nd[0], my_nd[1]};
    double v0lo, v[5] = {0.0, my_nd[2], my_nd[3], my_nd[4], my_nd[5]};
    const double* item_nd = s_nd[threadIdx.x >> 6][base];
    const double p0h = item_nd[kNd * kCheb], p0l = item_nd[kNd * kCheb + 1];
    const double peh = item_nd[kNd * (kCheb + 1)], pel = item_nd[kNd * (kCheb + 1) + 1];
    const dd span = dd_add(dd{peh, pel}, dd{-p0h, -p0l});
    const double rnb = nb > 1 ? 1.0 / (double)(nb - 1) : 0.0;
    const double B = (span.hi + span.lo) * rnb;    // R below is relative to this very B
    {
      const dd bm = two_prod(B, mk);
      const dd r = dd_add(dd_add(ph, dd{-p0h, -p0l}), dd{-bm.hi, -bm.lo});
      v[0] = r.hi;        // R at the node as a normalised double-double
      v0lo = r.lo;
    }
    // M-term integrands u |T+|^2, u |Tx|^2, u Re(T+ conj Tx), u Im(T+ conj Tx)
    // at this point, u from the smooth fit of its u-tile; usable when every
    // u-tile the item touches is fitted to within kUFitTol
    bool ufit = um.coef != nullptr && nb >= kMinInterp && nb <= kSsumMax;
    double gq[4], wq = 0.0, ures = 0.0;
    {
      // the channel's u-tiles follow those of the channels before it
      const int ub = ch * um.ntiles;
      const int ut0 = b0 / kUTile, ut1 = (b1 - 1) / kUTile;
      ufit = ufit && ut1 < um.ntiles &&
             (um.bad_prefix[ub + ut1 + 1] - um.bad_prefix[ub + ut0]) == 0;
      if (ufit && k < kCheb)   // largest fit residual over the item's u-tiles (the node lanes share the scan)
        for (int ut = ut0 + k; ut <= ut1; ut += kCheb) ures = fmax(ures, um.resid[ub + ut]);
      const double x = (double)b0 + mk;
      const int ut = min(max((int)(x * (1.0 / kUTile)), 0), max(um.ntiles - 1, 0));
      const double loc = 2.0 * (x - (double)ut * kUTile) / (double)(kUTile - 1) - 1.0;
      const double uu = um.coef ? cheb_eval10(um.coef + (int64_t)(ub + ut) * kUCoef, loc) : 0.0;
      gq[0] = uu * fma(v[1], v[1], v[2] * v[2]);
      gq[1] = uu * fma(v[3], v[3], v[4] * v[4]);
      gq[2] = uu * fma(v[1], v[3], v[2] * v[4]);
      gq[3] = uu * fma(v[2], v[3], -v[1] * v[4]);
      if (k < kCheb && um.ssum) {
        const int nq = min(nb, kSsumMax);
#pragma unroll
        for (int i = 0; i < 5; ++i) wq = fma(c_cheb_D[i][k], um.ssum[i * (kSsumMax + 1) + nq], wq);
      }
    }
    typedef RecLayout<MIXED> L;
    // Lane k forms sum_kn row[kn][k] v_kn: on node lanes (k < kCheb) the
    // interpolant's monomial coefficient k, on the end lanes its value at the
    // lane's own end point, which the lane has evaluated exactly.
    // FP64 path: R compensated (a twice-the-working-precision dot product:
    // error-free products and sums, their errors summed apart): R reaches a
    // few cycles, the node-to-monomial map has entries of a few hundred, and a
    // plain double sum would leave ~1e-13 cycles of cancellation error in the
    // coefficients.  Mixed path: a plain sum (its tolerance is 1e-9 cycles).
    double aRs = 0.0, aRx = 0.0, tmax = 0.0, gmax = 0.0, umax = 0.0;
    double aT[4], aTt[2][4], aG[4];
#pragma unroll
    for (int fn = 0; fn < 4; ++fn) {
      aT[fn] = 0.0; aG[fn] = 0.0; aTt[0][fn] = 0.0; aTt[1][fn] = 0.0;
    }
    __builtin_amdgcn_wave_barrier();
    my_nd[0] = v[0]; my_nd[1] = v0lo;
    my_nd[6] = gq[0]; my_nd[7] = gq[1]; my_nd[8] = gq[2]; my_nd[9] = gq[3];
    my_nd[10] = wq; my_nd[11] = ures;
    // the node's largest transfer component and |M-term integrand|
    my_nd[12] = fmax(fmax(fabs(v[1]), fabs(v[2])), fmax(fabs(v[3]), fabs(v[4])));
    my_nd[13] = fmax(fabs(gq[0]), fabs(gq[1]));
    __builtin_amdgcn_wave_barrier();
    // two nodes per pass (their LDS reads overlap); unrolled fully, the loop
    // hoists every node's table loads and needs more registers than the kernel
    // can hold at a useful occupancy
    // M-term integrands: lane 0 sums the quadrature, the end lanes interpolate
    const double sel0 = k == 0 ? 1.0 : 0.0, selE = k >= kCheb ? 1.0 : 0.0;
#pragma unroll 2
    for (int kn = 0; kn < kCheb; ++kn) {
      const double r9 = s_r9[kn][k];
      const double rT = MIXED ? s_rT[kn][k] : r9;
      const double2* nd = reinterpret_cast<const double2*>(item_nd + kNd * kn);
      const double2 n01 = nd[0], n23 = nd[1], n45 = nd[2], n67 = nd[3], n89 = nd[4], nab = nd[5],
                    ncd = nd[6];
      if constexpr (MIXED) {
        aRx = fma(n01.x, r9, aRx);
      } else {
        FSTAT_NO_CONTRACT
        const dd pr = two_prod(n01.x, r9);
        const dd sm = two_sum(aRs, pr.hi);
        aRs = sm.hi;
        aRx = fma(n01.y, r9, aRx + (sm.lo + pr.lo));
      }
      const double vt[4] = {n23.x, n23.y, n45.x, n45.y};
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) {
        aT[fn] = fma(vt[fn], rT, aT[fn]);
#pragma unroll
        for (int v2 = 0; v2 < (MIXED ? 1 : 2); ++v2)
          aTt[v2][fn] = fma(vt[fn], s_rt[v2][kn][k], aTt[v2][fn]);
      }
      tmax = fmax(tmax, ncd.x);
      gmax = fmax(gmax, ncd.y);
      umax = fmax(umax, nab.y);
      const double rg = fma(sel0, nab.x, selE * r9);
      const double gt[4] = {n67.x, n67.y, n89.x, n89.y};
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) aG[fn] = fma(gt[fn], rg, aG[fn]);
    }
    __builtin_amdgcn_wave_barrier();   // the slots are rewritten below
    const double cR = aRs + aRx;
    double d1 = 0.0, d2 = 0.0;         // sup |R'|, sup |R''| over the item (lane kCheb)
    if (sp.L > 0) {
      my_nd[0] = (double)k * fabs(cR);
      __builtin_amdgcn_wave_barrier();
      if (k == kCheb) {
#pragma unroll
        for (int kn = 1; kn < kCheb; ++kn) {
          const double a = item_nd[kNd * kn];
          d1 += a;
          d2 = fma((double)(kn - 1), a, d2);
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
    const double tolP = MIXED ? kInterpTolPhaseMixed : kInterpTolPhase;
    const double tolT = MIXED ? kInterpTolTMixed : kInterpTolT;
    bool bad = false;
    double err = 0.0;           // relative template error at this end point
    double errt[2] = {0.0, 0.0};   // transfer error of the degree-5 and -7 (mixed: 4) truncations
    double gerr = 0.0;          // M-term integrands' error (relative to max u |T|^2)
    if (k >= kCheb) {
      const double itmax = rcp_nr(tmax);      // the estimates below need no correct rounding
      // (aRs - v0 is exact wherever the interpolant is close enough to pass)
      const double dph = fabs(((aRs - v[0]) + aRx) - v0lo);
      bad = !(dph <= tolP);
      err = 2.0 * kPi * dph;
#pragma unroll
      for (int fn = 1; fn < 5; ++fn) {
        const double d = fabs(aT[fn - 1] - v[fn]);
        bad = bad || !(d <= tolT * tmax);
        err = fmax(err, d * itmax);
#pragma unroll
        for (int v2 = 0; v2 < (MIXED ? 1 : 2); ++v2)
          errt[v2] = fmax(errt[v2], fabs(aTt[v2][fn - 1] - v[fn]) * itmax);
      }
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) gerr = fmax(gerr, fabs(aG[fn] - gq[fn]));
      gerr = gmax > 0.0 ? gerr * rcp_nr(gmax) : (gerr > 0.0 ? 1.0 : 0.0);
    }
    const double tolG = MIXED ? kInterpTolTMixed : 4.0 * kInterpTolT;
    const uint64_t gbadmask = __ballot(k >= kCheb && !(gerr <= tolG));
    gerr = fmax(fmax(gerr, __shfl(gerr, base + kCheb + 1, 64)), umax);
    const uint64_t badmask = __ballot(bad);
    err = fmax(__shfl(err, base + kCheb, 64), __shfl(err, base + kCheb + 1, 64));
    double gsum[4];
#pragma unroll
    for (int fn = 0; fn < 4; ++fn) gsum[fn] = __shfl(aG[fn], base, 64);
    // FP64: lowest transfer degree whose truncation error stays within the
    // item's own interpolation error, or kTruncFloor of the largest component
    // (a larger allowance sends more items of ill-conditioned partitions to
    // the exact re-evaluation than the lower degree saves)
    int degT = MIXED ? kDegT : kCheb - 1;
    if constexpr (!MIXED) {
      const double allow = fmin(fmax(err, kTruncFloor), tolT);
      const double e7 = fmax(__shfl(errt[1], base + kCheb, 64), __shfl(errt[1], base + kCheb + 1, 64));
      const double e5 = fmax(__shfl(errt[0], base + kCheb, 64), __shfl(errt[0], base + kCheb + 1, 64));
      if (e5 <= allow) { degT = 5; err = fmax(err, e5); }
      else if (e7 <= allow) { degT = 7; err = fmax(err, e7); }
    } else {
      const double e4 = fmax(__shfl(errt[0], base + kCheb, 64), __shfl(errt[0], base + kCheb + 1, 64));
      if (e4 <= tolT) { degT = kDegTLow; err = fmax(err, e4); }
    }
    const bool mine = lane - base < kLanesItem && grp * kItemsWave + q < W;   // not a repeat lane
    if (!mine) continue;
    const bool mq = ufit && ((gbadmask >> base) & ((1ull << kLanesItem) - 1ull)) == 0ull;
    // items without quadrature M-terms (u not fitted on one of their u-tiles,
    // or M-term interpolants that miss an end point) go to the exact loop too
    const bool rej = nb < kMinInterp || !mq ||
                     ((badmask >> base) & ((1ull << kLanesItem) - 1ull)) != 0ull;
    if (mq && k < 4)
      partials[(int64_t)w * 8 + 4 + k] = k == 0 ? gsum[0] : (k == 1 ? gsum[1] : (k == 2 ? gsum[2] : gsum[3]));
    double* r = rec + (int64_t)w * kRec;
    if (k < kCheb) {
      r[k] = cR;
      if (k < L::nT) {
#pragma unroll
        for (int fn = 1; fn < 5; ++fn)
          r[kCheb + (fn - 1) * L::nT + k] =
              MIXED ? (degT == kDegTLow ? aTt[0][fn - 1] : aT[fn - 1])
                    : (degT == 5 ? aTt[0][fn - 1] : (degT == 7 ? aTt[1][fn - 1] : aT[fn - 1]));
      }
    } else if (k == kCheb) {
      FSTAT_NO_CONTRACT
      const double alpha = 2.0 * rnb;
      r[L::tail] = (p0h - floor(p0h)) + p0l;     // fractional cycle at the first bin
      r[L::tail + 1] = B - rint(B);              // whole cycles per bin drop out (m is an integer)
      r[L::tail + 2] = B;
      bool blocks = false;
      if (sp.L > 0) {
        const double half = 0.5 * (double)(sp.L - 1) * alpha;
        const double sl = alpha * d1;
        blocks = kPi * d2 * half * half <= sp.psi && B - sl >= -sp.hq && B + sl <= sp.smax + sp.hq &&
                 bin_freq(g, b1 - 1) < sp.fmax;
      }
      const int state = rej ? kRecExact : (blocks ? kRecBlocks : kRecBins);
      int2* ri = reinterpret_cast<int2*>(r + L::tail + 3);
      ri[0] = make_int2(state | degT << 8 | ch << 16, b0);
      ri[1] = make_int2(nb, 0);
      r[L::tail + 5] = alpha;
      r[L::tail + 6] = -B / g.df;
      xflag[w] = rej ? kItemExact : (blocks ? kItemBlocks : kItemBins);
      // the template error times the norm sqrt(sum u) max|T| of the item's
      // templates, and the M-term quadrature's error bound: its relative error
      // at the end points times max u |T|^2 times the bin count (see k_mark)
      const int64_t uo = (int64_t)ch * (g.nbins + 1);
      const double U = um.upre ? fmax(um.upre[uo + b1] - um.upre[uo + b0], 0.0) : (double)nb;
      xerr[w] = make_float2((float)(err * tmax * __builtin_amdgcn_sqrt(U)), mq ? (float)(gerr * gmax * nb) : 0.0f);
      if (rej) direct[atomicAdd(ndirect, 1)] = w;
    }
  }
}

// The bins of the interpolated items, tile by tile: the tile's w is staged
// once in LDS; each wave takes one item at a time, broadcasts its record into
// registers and runs the per-bin loop from LDS.
template <bool MIXED>
__global__ __launch_bounds__(256) void k_eval_interp(Grid g,
                                                     Tiling tl,
                                                     const int32_t* __restrict__ tile_items,
                                                     const int32_t* __restrict__ tile_off,
                                                     const int32_t* __restrict__ unit_off,
                                                     int32_t ntiles,
                                                     int32_t* __restrict__ tile_ctr,
                                                     const double* __restrict__ wr64,
                                                     const double* __restrict__ wi64,
                                                     const float* __restrict__ wr32,
                                                     const float* __restrict__ wi32,
                                                     double* __restrict__ rec,
                                                     double* __restrict__ partials) {
  typedef typename std::conditional<MIXED, float, double>::type DT;
  extern __shared__ unsigned char smem[];
  // The tile's w (and on the FP64 path e_j) at a fixed stride of the largest
  // tile, so that every per-bin read shares one address register (constant
  // offsets) whatever the tile size.  Every item here has its M-terms from the
  // node kernel's quadrature (the others go to the exact loop), so u is not
  // staged; e_j is kept in FP32 (|e_j| <= half an ulp of f_j; its product with
  // t_f <~ 1e8 s enters the phase at <~ 1e-10 cycles, and FP32 rounding of it
  // at ~1e-17 cycles).  FP64: 20 B per bin, three blocks of 2560-bin tiles per
  // CU.
  constexpr int TS = MIXED ? kMaxTileMixed : kMaxTileFp64;
  const double2* s_tab = c_sincos;                       // FP64 loop: sin, cos table
  DT* s_wr = reinterpret_cast<DT*>(smem);
  DT* s_wi = s_wr + TS;
  float* s_e = reinterpret_cast<float*>(s_wi + TS);      // FP64 loop: grid rounding e_j
  __shared__ int s_unit[3];                       // tile, first item, item count
  __shared__ double s_rec[4][64];                // each wave's current item record
  const DT* gwr;
  const DT* gwi;
  if constexpr (MIXED) { gwr = wr32; gwi = wi32; }
  else { gwr = wr64; gwi = wi64; }
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int nwv = blockDim.x >> 6;
  const int nunits = unit_off[ntiles];
  if (nunits == 0) return;
  // The current unit: its items, the channel's data offset, and the bins of its
  // tile (of all tiles its items may reach) not yet staged.  More than the LDS stage go through it in parts; a wave
  // takes the same items in each and adds to their sums.
  int i0 = 0, cnt = 0, j0 = 0, j_end = 0;
  int64_t co = 0;
  for (;; j0 += TS) {
    if (j0 >= j_end) {
      // next unit (dynamic): up to kUnitItems items of one tile
      if (threadIdx.x == 0) {
        const int u = atomicAdd(tile_ctr, 1);
        int t = -1, first = 0, count = 0;
        if (u < nunits) {
          int lo = 0, hi = ntiles;                   // last tile with unit_off[t] <= u
          while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (unit_off[mid] <= u) lo = mid; else hi = mid;
          }
          t = lo;
          first = tile_off[t] + (u - unit_off[t]) * kUnitItems;
          count = min(kUnitItems, tile_off[t + 1] - first);
        }
        s_unit[0] = t; s_unit[1] = first; s_unit[2] = count;
      }
      __syncthreads();
      const int tx = s_unit[0];
      if (tx < 0) break;
      // tiles of all channels are numbered channel by channel
      const int tch = tx / tl.ntiles;
      co = (int64_t)tch * g.nbins;
      i0 = s_unit[1];
      cnt = s_unit[2];
      j0 = (tx - tch * tl.ntiles) * tl.T;
      j_end = (int)min((int64_t)j0 + (int64_t)tl.mmax * tl.T, g.nbins);
    }
    const int nt = min(TS, j_end - j0);
    for (int i = threadIdx.x; i < nt; i += blockDim.x) {
      s_wr[i] = gwr[co + j0 + i];
      s_wi[i] = gwi[co + j0 + i];
      if constexpr (!MIXED) {
        // f_j = (k_lo + j) df rounds to a double; e_j is the rounding error of
        // that product (one FMA), formed once per bin of the tile
        const double jd = (double)(g.k_lo + j0 + i);
        s_e[i] = (float)fma(jd, g.df, -(jd * g.df));
      }
    }
    __syncthreads();
    typedef RecLayout<MIXED> L;
    double* R = s_rec[wv];
    // Each item's record holds all the loop needs of it; a wave loads the next
    // item's record while it runs the current one, so that only the first
    // load of a unit is waited for.
    int wn = wv < cnt ? tile_items[i0 + wv] : 0;
    double rv = (wv < cnt && lane < kRec) ? rec[(int64_t)wn * kRec + lane] : 0.0;
    for (int idx = wv; idx < cnt; idx += nwv) {
      const int w = wn;
      // the record through the wave's LDS slot: one write, then broadcast reads
      // (LDS operations of one wave complete in order)
      if (lane < kRec) R[lane] = rv;
      __builtin_amdgcn_wave_barrier();
      const int idn = idx + nwv;
      wn = idn < cnt ? tile_items[i0 + idn] : 0;
      rv = (idn < cnt && lane < kRec) ? rec[(int64_t)wn * kRec + lane] : 0.0;
      const int b0 = rec_int(R[L::tail + 3], 1);
      const int e0 = max(b0 - j0, 0);             // LDS offset of the item's first bin here
      const int mo = e0 + j0 - b0;                // that bin's number in the item
      const int nb = min(b0 + rec_int(R[L::tail + 4], 0), j0 + nt) - (b0 + mo);   // bins here
      if (nb <= 0) {
        __builtin_amdgcn_wave_barrier();
        continue;
      }
      double cR[kCheb];
#pragma unroll
      for (int n = 0; n < kCheb; ++n) cR[n] = R[n];
      const double A = R[L::tail];
      const double Bp = R[L::tail + 1];
      const int flags = rec_int(R[L::tail + 3], 0);
      const int degT = (flags >> 8) & 255;        // transfer degree
      const double alpha = R[L::tail + 5];        // 2 / (nb - 1)
      if constexpr (!MIXED) {
        // The grid is f_j = (k_lo + j) df rounded to a double; the interpolants
        // are exact in f, so the phase moves by (dPhi/df)(f_j - exact) =
        // -(B / df) e_j, with e_j the rounding error of the product (staged
        // with the tile): up to ~1e-9 cycles at t_f ~ 1e8 s.
        const double kB = R[L::tail + 6];           // -B / df
        // Difference recurrence for items whose lanes get runs of at least
        // kRecMinRun bins.  Lane l takes the contiguous bins m0 = l Lr ..
        // m0 + Lr - 1 (Lr odd, so that the lanes' LDS addresses fall in
        // distinct banks).  With a_k = alpha^k R^(k)(s0) / k! the phase is
        // Phi(m0 + t) = Phi(m0) + Bp t + sum_k a_k t^k; its forward differences
        // D_j (D_j(t + 1) = D_j(t) + D_{j+1}(t)) start at D_1 = Bp + sum_k a_k
        // and D_j = sum_k j! S(k, j) a_k (S: Stirling numbers of the second
        // kind).  Per bin the template factor advances as E0 <- E0 E1(t), with
        // E1(t) = E1(0) e^{i phi(t)} and phi(t) = 2 pi sum_{i<t} D_2(i) (D_2, D_3
        // advanced by their differences, D_4 held): no phase polynomial and no
        // sine per bin.  Over <= 33 bins the rounding of the products stays
        // near 1e-14, below the direct evaluation's own ~1e-13 cycles; an item
        // takes the direct loop when phi can leave the range of its series or
        // the neglected D_5 could move the phase by more than kRecTrunc.
        const int Lr = ((nb + 63) >> 6) | 1;
        const int r0 = lane * Lr;                 // the run's first bin here, in the item
        const int m0 = mo + r0;
        const int cnt = min(max(nb - r0, 0), Lr);
        double E0r = 0.0, E0i = 0.0, E1r = 0.0, E1i = 0.0, th2 = 0.0, th3 = 0.0, th4 = 0.0;
        bool use_rec = Lr >= kRecMinRun;
        if (use_rec) {
          const double s0 = fma(alpha, (double)m0, -1.0);
          // Taylor coefficients of R at s0 (repeated synthetic division)
          double p[kCheb];
#pragma unroll
          for (int n = 0; n < kCheb; ++n) p[n] = cR[n];
#pragma unroll
          for (int k = 0; k < kCheb - 1; ++k)
#pragma unroll
            for (int j = kCheb - 2; j >= k; --j) p[j] = fma(p[j + 1], s0, p[j]);
          double ap[kCheb];
          ap[0] = 1.0;
#pragma unroll
          for (int k = 1; k < kCheb; ++k) ap[k] = ap[k - 1] * alpha;
          double d1 = 0.0, d2 = 0.0, d3 = 0.0, d4 = 0.0, d5 = 0.0;
#pragma unroll
          for (int k = kCheb - 1; k >= 1; --k) {    // smallest terms first
            const double ak = p[k] * ap[k];
            d1 += ak;
            if (k >= 2) d2 = fma(kStirF[k][2], ak, d2);
            if (k >= 3) d3 = fma(kStirF[k][3], ak, d3);
            if (k >= 4) d4 = fma(kStirF[k][4], ak, d4);
            if (k >= 5) d5 = fma(kStirF[k][5], ak, d5);
          }
          d1 += Bp;
          sincos_tab(fma(Bp, (double)m0, p[0]) + A, s_tab, E0i, E0r);
          sincos_tab(d1, s_tab, E1i, E1r);
          th2 = kTwoPi * d2;
          th3 = kTwoPi * d3;
          th4 = kTwoPi * d4;
          const double x = (double)Lr;
          const double phimax = x * (fabs(th2) + x * (fabs(th3) + x * fabs(th4)));
          const double c5 = x * (x - 1.0) * (x - 2.0) * (x - 3.0) * (x - 4.0) * (1.0 / 120.0);
          const bool ok = cnt == 0 || (phimax <= kRecPhiMax && c5 * kTwoPi * fabs(d5) <= kRecTrunc);
          use_rec = __all(ok);
        }
        if (lane == 0 && use_rec)                      // for fstat_interp_stats
          *reinterpret_cast<int*>(rec + (int64_t)w * kRec + L::tail + 3) =
              (flags & ~255) | kRecBinsShort;
        // DT: degree of the transfer interpolants (5, 7 or 9)
        auto loop = [&](auto dt) {
          constexpr int DT = decltype(dt)::value;
          int idx;
          {
            // N-terms only.  They are linear in the transfer interpolants
            // T(s) = sum_k c_k s^k, so the loop sums the moments
            // sum_j w_j e^{i Phi_j} s_j^k (k <= DT) and the coefficients are
            // applied once per lane afterwards: no transfer polynomial per bin.
            double mr[DT + 1], mm[DT + 1];
            using First = std::true_type;
            using Next = std::false_type;
            if (use_rec) {
              // The run's bins are equally spaced in s, so the loop sums
              // binomial moments instead: per bin A_m += A_{m-1} (m = DT..1),
              // then A_0 += X_t, which leaves A_m = sum_t X_t C(cnt - 1 - t, m)
              // (X_t = w e^{i Phi} at the run's bin t); no power of s per bin.
              // They become power moments once per lane below.
              const double kBe = kTwoPi * kB;
              double phi = 0.0, t2 = th2, t3 = th3;
              double er = E0r, ei = E0i;
              auto rec_bin = [&](auto first, double a, double b, float ef) {
                constexpr bool F = decltype(first)::value;
                // the grid rounding as the factor 1 + i eps (|eps| <~ 1e-8)
                const double eps = kBe * (double)ef;
                const double xr = fma(-eps, ei, er), xi = fma(eps, er, ei);
                if constexpr (F) {
                  mr[0] = fma(-b, xi, a * xr);
                  mm[0] = fma(b, xr, a * xi);
#pragma unroll
                  for (int m = 1; m <= DT; ++m) mr[m] = mm[m] = 0.0;
                } else {
#pragma unroll
                  for (int m = DT; m >= 1; --m) {
                    mr[m] += mr[m - 1];
                    mm[m] += mm[m - 1];
                  }
                  mr[0] = fma(a, xr, fma(-b, xi, mr[0]));
                  mm[0] = fma(a, xi, fma(b, xr, mm[0]));
                }
                // E1(t) = E1(0) e^{i phi}: |phi| <= kRecPhiMax, series to phi^6
                // (cos) and phi^5 (sin), remainders below 1e-17
                const double z = phi * phi;
                const double cph = fma(fma3(1.0 / 24.0, z, -0.5), z, 1.0);
                const double sph = phi * fma(fma3(1.0 / 120.0, z, -1.0 / 6.0), z, 1.0);
                const double e1r = E1r * cph - E1i * sph, e1i = E1r * sph + E1i * cph;
                const double nr = er * e1r - ei * e1i;
                ei = er * e1i + ei * e1r;
                er = nr;
                phi += t2;
                t2 += t3;
                t3 += th4;
              };
              // the first bin sets the moments (lanes without bins take w = 0);
              // the rest of an odd run goes two bins per pass
              const int ib = e0 + r0;
              const bool any = cnt > 0;
              rec_bin(First{}, any ? s_wr[ib] : 0.0, any ? s_wi[ib] : 0.0, any ? s_e[ib] : 0.0f);
              int t = 1;
              for (; t + 1 < cnt; t += 2) {
                const double a1 = s_wr[ib + t], a2 = s_wr[ib + t + 1];
                const double b1 = s_wi[ib + t], b2 = s_wi[ib + t + 1];
                const float f1 = s_e[ib + t], f2 = s_e[ib + t + 1];
                rec_bin(Next{}, a1, b1, f1);
                rec_bin(Next{}, a2, b2, f2);
              }
              if (t < cnt) rec_bin(Next{}, s_wr[ib + t], s_wi[ib + t], s_e[ib + t]);
              // To power moments M_k = sum_t X_t s_t^k.  With u = cnt - 1 - t,
              // s_t = s_e - alpha u (s_e: the run's last bin): sum_t X_t u^j =
              // sum_m m! S(j, m) A_m, scaled by (-alpha)^j, then shifted to the
              // origin by M_k = sum_j C(k, j) s_e^(k - j) (...)_j.  Over a run
              // of <~ 0.03 in s every step keeps its terms near the result's
              // own size.
#pragma unroll
              for (int j = DT; j >= 2; --j) {
                double pr = kStirF[j][j] * mr[j], pi = kStirF[j][j] * mm[j];
#pragma unroll
                for (int m = j - 1; m >= 2; --m) {
                  pr = fma(kStirF[j][m], mr[m], pr);
                  pi = fma(kStirF[j][m], mm[m], pi);
                }
                mr[j] = pr + mr[1];
                mm[j] = pi + mm[1];
              }
              const double na = -alpha;
              double pw = na;
#pragma unroll
              for (int j = 1; j <= DT; ++j) {
                mr[j] *= pw;
                mm[j] *= pw;
                pw *= na;
              }
              const double se = fma(alpha, (double)(m0 + cnt - 1), -1.0);
#pragma unroll
              for (int k = 0; k < DT; ++k)
#pragma unroll
                for (int j = DT; j > k; --j) {
                  mr[j] = fma(se, mr[j - 1], mr[j]);
                  mm[j] = fma(se, mm[j - 1], mm[j]);
                }
            } else {
              // direct form: even moments from W = w e^{i Phi}, odd ones from
              // W s, both against even powers of s
              auto moments = [&](double Wr, double Wi, double s, double s2, double s4, double s8) {
                const double Vr = Wr * s, Vi = Wi * s;
                const double pe[5] = {1.0, s2, s4, s4 * s2, s8};
                mr[0] += Wr;
                mm[0] += Wi;
                mr[1] += Vr;
                mm[1] += Vi;
#pragma unroll
                for (int k = 2; k <= DT; ++k) {
                  const double xr = (k & 1) ? Vr : Wr, xi = (k & 1) ? Vi : Wi;
                  mr[k] = fma(xr, pe[k >> 1], mr[k]);
                  mm[k] = fma(xi, pe[k >> 1], mm[k]);
                }
              };
              auto one_bin = [&](int mi, double a, double b, double ej) {
                const double m = (double)(mo + mi);
                const double s = fma(alpha, m, -1.0);
                const double s2 = s * s, s4 = s2 * s2, s8 = s4 * s4;
                const double ph = fma(Bp, m, estrin9(cR, s, s2, s4, s8)) + fma(kB, ej, A);
                double sps, cps;
                sincos_tab(ph, s_tab, sps, cps);
                moments(a * cps - b * sps, a * sps + b * cps, s, s2, s4, s8);
              };
#pragma unroll
              for (int k = 0; k <= DT; ++k) mr[k] = mm[k] = 0.0;
              // lanes interleaved; two bins per pass (half the loop control per
              // bin), then at most one left over per lane
              int mi = lane;
              for (; mi + 64 < nb; mi += 128) {
                const int i1 = e0 + mi, i2 = i1 + 64;
                const double a1 = s_wr[i1], b1 = s_wi[i1], e1 = s_e[i1];
                const double a2 = s_wr[i2], b2 = s_wi[i2], e2 = s_e[i2];
                one_bin(mi, a1, b1, e1);
                one_bin(mi + 64, a2, b2, e2);
              }
              if (mi < nb) {
                const int i1 = e0 + mi;
                one_bin(mi, s_wr[i1], s_wi[i1], s_e[i1]);
              }
            }
            // sum Wr T+r + Wi T+i, sum Wi T+r - Wr T+i, and the same for x: FMA
            // chains, one transfer component pair at a time (fewer live registers)
            double acc[4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
              for (int k = 0; k <= DT; ++k) {
                const double tr = R[kCheb + 2 * h * L::nT + k], ti = R[kCheb + (2 * h + 1) * L::nT + k];
                acc[2 * h] = fma(tr, mr[k], k ? fma(ti, mm[k], acc[2 * h]) : ti * mm[k]);
                acc[2 * h + 1] = fma(tr, mm[k], k ? fma(-ti, mr[k], acc[2 * h + 1]) : -ti * mr[k]);
              }
            }
            __builtin_amdgcn_wave_barrier();   // the slot is rewritten for the next item
            const double tot = wave_sum4(acc, lane, idx);
            if ((lane & 15) == 0) {
              double* o = partials + (int64_t)w * 8 + idx;
              *o = mo > 0 ? *o + tot : tot;
            }
          }
        };
        using D5 = std::integral_constant<int, 5>;
        using D7 = std::integral_constant<int, 7>;
        using D9 = std::integral_constant<int, 9>;
        if (degT == 5) loop(D5{});
        else if (degT == 7) loop(D7{});
        else loop(D9{});
      } else {
        // Lane l takes the contiguous bins m0 = l Lr .. m0 + Lr - 1 (Lr odd:
        // distinct LDS banks).  The phase R(s) + Bp m + A [turns] advances by
        // its forward differences in FP64: R has degree 9, so the ninth
        // difference is constant and every phase of the run is exact up to
        // rounding (~1e-13 turns over a run), no polynomial per bin; where a
        // bound on what the fifth to ninth differences add stays below
        // kMixTrunc on every lane's run, the wave holds the fourth constant
        // and forms only the first four.  The
        // N-terms are summed in FP32 as binomial moments (A_m += A_{m-1}, then
        // A_0 += w e^{i Phi}: A_m = sum_t w_t e^{i Phi_t} C(cnt - 1 - t, m)),
        // changed once per lane to power moments sum w e^{i Phi} s^k (k <= D)
        // over the run's <~ 0.03 in s, where each step keeps its terms near the
        // result's size; their FP32 rounding, ~1e-7 relative, is far inside the
        // mixed path's bar.  The transfer degree is kDegT, or kDegTLow where the
        // node kernel found it enough; the coefficients are applied in FP64.
        const int Lr = ((nb + 63) >> 6) | 1;
        const int r0 = lane * Lr;                 // the run's first bin here, in the item
        const int m0 = mo + r0;
        const int cnt = min(max(nb - r0, 0), Lr);
        double dd[kCheb];                 // dd[j]: j-th forward difference (j >= 1)
        double ph;
        bool trunc;
        {
          // Taylor coefficients of R at the run's start (repeated synthetic
          // division), a_k = alpha^k R^(k)(s0) / k!, D_j = sum_k j! S(k, j) a_k
          const double s0 = fma(alpha, (double)m0, -1.0);
          double p[kCheb];
#pragma unroll
          for (int n = 0; n < kCheb; ++n) p[n] = cR[n];
#pragma unroll
          for (int k = 0; k < kCheb - 1; ++k)
#pragma unroll
            for (int j = kCheb - 2; j >= k; --j) p[j] = fma(p[j + 1], s0, p[j]);
          // What the fifth to ninth differences add to the phase t bins in:
          // sum_{k>=5} a_k sum_{j>=5} C(t, j) j! S(k, j), whose inner sums are
          // at most sum_j C(t, j) j! S(k, j) = t^k; so with t < Lr it is below
          // sum_{k>=5} |R^(k)(s0) / k!| (alpha Lr)^k.
          const double x = alpha * (double)Lr;
          double xk = (x * x) * (x * x), bound = 0.0;
#pragma unroll
          for (int k = kMixDiff + 1; k < kCheb; ++k) {
            xk *= x;
            bound = fma(fabs(p[k]), xk, bound);
          }
          trunc = __all(cnt == 0 || bound <= kMixTrunc);
          double ap[kCheb];
          ap[1] = alpha;
#pragma unroll
          for (int k = 2; k < kCheb; ++k) ap[k] = ap[k - 1] * alpha;
#pragma unroll
          for (int j = 1; j < kCheb; ++j) dd[j] = 0.0;
#pragma unroll
          for (int k = kCheb - 1; k >= 1; --k) {    // smallest terms first
            const double ak = p[k] * ap[k];
#pragma unroll
            for (int j = 1; j <= k && j <= kMixDiff; ++j) dd[j] = fma(kStirF[k][j], ak, dd[j]);
          }
          if (!trunc) {                               // the wave carries all nine
#pragma unroll
            for (int k = kCheb - 1; k > kMixDiff; --k) {
              const double ak = p[k] * ap[k];
#pragma unroll
              for (int j = kMixDiff + 1; j <= k; ++j) dd[j] = fma(kStirF[k][j], ak, dd[j]);
            }
          }
          dd[1] += Bp;
          ph = fma(Bp, (double)m0, p[0]) + A;
          ph -= rint(ph);
        }
        if (lane == 0 && trunc)                        // for fstat_interp_stats
          *reinterpret_cast<int*>(rec + (int64_t)w * kRec + L::tail + 3) =
              (flags & ~255) | kRecBinsShort;
        // D: transfer degree; ND: forward differences carried (the last held)
        auto loop = [&](auto dt, auto ndt) {
          constexpr int D = decltype(dt)::value;
          constexpr int ND = decltype(ndt)::value;
          int idx;
          float mr[D + 1], mm[D + 1];
          auto bin = [&](auto first, float a, float b) {
            constexpr bool F = decltype(first)::value;
            const float rf = (float)(ph - rint(ph));
            const float sps = __builtin_amdgcn_sinf(rf), cps = __builtin_amdgcn_cosf(rf);
            if constexpr (F) {
              mr[0] = fmaf(-b, sps, a * cps);
              mm[0] = fmaf(b, cps, a * sps);
#pragma unroll
              for (int m = 1; m <= D; ++m) mr[m] = mm[m] = 0.0f;
            } else {
#pragma unroll
              for (int m = D; m >= 1; --m) {
                mr[m] += mr[m - 1];
                mm[m] += mm[m - 1];
              }
              mr[0] = fmaf(a, cps, fmaf(-b, sps, mr[0]));
              mm[0] = fmaf(a, sps, fmaf(b, cps, mm[0]));
            }
            ph += dd[1];
#pragma unroll
            for (int j = 1; j < ND; ++j) dd[j] += dd[j + 1];
          };
          using First = std::true_type;
          using Next = std::false_type;
          // the first bin sets the moments (lanes without bins take w = 0);
          // the rest of an odd run goes two bins per pass
          const int ib = e0 + r0;
          const bool any = cnt > 0;
          bin(First{}, any ? s_wr[ib] : 0.0f, any ? s_wi[ib] : 0.0f);
          int t = 1;
          for (; t + 1 < cnt; t += 2) {
            const float a1 = s_wr[ib + t], a2 = s_wr[ib + t + 1];
            const float b1 = s_wi[ib + t], b2 = s_wi[ib + t + 1];
            bin(Next{}, a1, b1);
            bin(Next{}, a2, b2);
          }
          if (t < cnt) bin(Next{}, s_wr[ib + t], s_wi[ib + t]);
          // to power moments: with u = cnt - 1 - t and s_t = s_e - alpha u,
          // sum_t X_t u^j = sum_m m! S(j, m) A_m, scaled by (-alpha)^j, then
          // shifted to the origin by M_k = sum_j C(k, j) s_e^(k - j) (...)_j
#pragma unroll
          for (int j = D; j >= 2; --j) {
            float pr = (float)kStirF[j][j] * mr[j], pi = (float)kStirF[j][j] * mm[j];
#pragma unroll
            for (int m = j - 1; m >= 2; --m) {
              pr = fmaf((float)kStirF[j][m], mr[m], pr);
              pi = fmaf((float)kStirF[j][m], mm[m], pi);
            }
            mr[j] = pr + mr[1];
            mm[j] = pi + mm[1];
          }
          const float na = (float)(-alpha);
          float pw = na;
#pragma unroll
          for (int j = 1; j <= D; ++j) {
            mr[j] *= pw;
            mm[j] *= pw;
            pw *= na;
          }
          const float se = (float)fma(alpha, (double)(m0 + cnt - 1), -1.0);
#pragma unroll
          for (int k = 0; k < D; ++k)
#pragma unroll
            for (int j = D; j > k; --j) {
              mr[j] = fmaf(se, mr[j - 1], mr[j]);
              mm[j] = fmaf(se, mm[j - 1], mm[j]);
            }
          double red[4];
#pragma unroll
          for (int k = 0; k <= D; ++k) {
            const double t0 = R[kCheb + k], t1 = R[kCheb + L::nT + k];
            const double t2 = R[kCheb + 2 * L::nT + k], t3 = R[kCheb + 3 * L::nT + k];
            const double r = mr[k], q = mm[k];
            red[0] = fma(t0, r, k ? fma(t1, q, red[0]) : t1 * q);
            red[1] = fma(t0, q, k ? fma(-t1, r, red[1]) : -t1 * r);
            red[2] = fma(t2, r, k ? fma(t3, q, red[2]) : t3 * q);
            red[3] = fma(t2, q, k ? fma(-t3, r, red[3]) : -t3 * r);
          }
          __builtin_amdgcn_wave_barrier();   // the slot is rewritten for the next item
          const double tot = wave_sum4(red, lane, idx);
          if ((lane & 15) == 0) {
            double* o = partials + (int64_t)w * 8 + idx;
            *o = mo > 0 ? *o + tot : tot;
          }
        };
        using DLow = std::integral_constant<int, kDegTLow>;
        using DHigh = std::integral_constant<int, kDegT>;
        using NShort = std::integral_constant<int, kMixDiff>;
        using NFull = std::integral_constant<int, kCheb - 1>;
        if (degT == kDegTLow) {
          if (trunc) loop(DLow{}, NShort{});
          else loop(DLow{}, NFull{});
        } else {
          if (trunc) loop(DHigh{}, NShort{});
          else loop(DHigh{}, NFull{});
        }
      }
    }
    __syncthreads();   // every wave is done with this stage's LDS and s_unit
  }
}

// ---------------------------------------------------------------------------
// the block loop: items evaluated from the plan's block spectra
// ---------------------------------------------------------------------------
// largest curvature over a block [rad] (see spectra.hip)
constexpr double kSpecPsiFp64 = 0.25;
constexpr double kSpecPsiMixed = 1.0;
constexpr int kGrp = kSpecNodes;        // lanes per item: one per node of a block's row
constexpr int kRecPad = 58;             // record stride in LDS: the four records of a wave
                                        // in distinct banks
constexpr int kBlkAhead = 2;            // rows of the spectra in flight per lane
static_assert(kRec <= kRecPad && kGrp == 16, "group layout");

// lane n of each row of 16 to the whole row
template <int N>
__device__ __forceinline__ double row_bcast(double x) {
  int2 v = *reinterpret_cast<int2*>(&x);
  v.x = __builtin_amdgcn_mov_dpp(v.x, 0x150 + N, 0xf, 0xf, true);   // row_newbcast
  v.y = __builtin_amdgcn_mov_dpp(v.y, 0x150 + N, 0xf, 0xf, true);
  return *reinterpret_cast<double*>(&v);
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
  int2 v = *reinterpret_cast<int2*>(&x);
  v.x = __builtin_amdgcn_mov_dpp(v.x, CTRL, 0xf, 0xf, true);
  v.y = __builtin_amdgcn_mov_dpp(v.y, CTRL, 0xf, 0xf, true);
  return x + *reinterpret_cast<double*>(&v);
}
// sum over each row of 16 lanes, on every lane (fixed order)
__device__ __forceinline__ double row_sum(double x) {
  x = dpp_add<0xB1>(x);                 // quad_perm [1, 0, 3, 2]
  x = dpp_add<0x4E>(x);                 // quad_perm [2, 3, 0, 1]
  x = dpp_add<0x141>(x);                // row_half_mirror
  return dpp_add<0x140>(x);             // row_mirror
}

// largest of a value that is the same in each row of 16 lanes, for the whole wave
__device__ __forceinline__ int row_max(int x) {
  return max(max(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             max(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
// x (|x| < 2^31) rounded to a whole number, as a double and an integer, by an addition
// that leaves the number in the low bits
__device__ __forceinline__ double round_int(double x, double scale, int& n) {
  const double big = 6755399441055744.0;                 // 1.5 2^52
  const double t = fma(x, scale, big);
  n = __double2loint(t);
  return t - big;
}

// An item's per-lane sums sum_j V_j s_j^k of the samples V = S e^{i Phi} that its
// sixteen lanes take (nodes of its whole blocks, or bins of its partial ones),
// s in [-1, 1] the item's coordinate.  DT: highest power.  FP64: even moments
// from V, odd ones from V s, against even powers of s.
template <bool MIXED, int DT>
struct Moments {
  typedef typename std::conditional<MIXED, float, double>::type T;
  T mr[DT + 1], mm[DT + 1];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k <= DT; ++k) mr[k] = mm[k] = T(0);
  }
  // ph: the sample's phase [turns]; (a, b): its data
  __device__ __forceinline__ void add(double ph, double sd, T a, T b, const double2* tab) {
    T sp, cp;
    if constexpr (MIXED) {
      const float rf = (float)(ph - rint(ph));
      sp = __builtin_amdgcn_sinf(rf);
      cp = __builtin_amdgcn_cosf(rf);
    } else {
      // sincos_tab with the rounding of round_int
      int n;
      const double nd = round_int(ph, (double)kSinTab, n);
      const double2 e = tab[n & (kSinTab - 1)];
      const double th = fma(-1.0 / (double)kSinTab, nd, ph) * 6.283185307179586477;
      const double z = th * th;
      const double ps = fma3(1.0 / 120.0, z, -1.0 / 6.0);
      const double pc = fma(fma3(-1.0 / 720.0, z, 1.0 / 24.0), z, -0.5);
      const double sl = fma(th * z, ps, th), cl = fma(z, pc, 1.0);
      sp = fma(e.x, cl, e.y * sl);
      cp = fma(e.y, cl, -(e.x * sl));
    }
    const T s = (T)sd, s2 = s * s;
    const T Vr = a * cp - b * sp, Vi = a * sp + b * cp;
    const T Ur = Vr * s, Ui = Vi * s;
    mr[0] += Vr;
    mm[0] += Vi;
    mr[1] += Ur;
    mm[1] += Ui;
    T pw = s2;
#pragma unroll
    for (int k = 2; k <= DT; ++k) {
      const T xr = (k & 1) ? Ur : Vr, xi = (k & 1) ? Ui : Vi;
      mr[k] = fma(xr, pw, mr[k]);
      mm[k] = fma(xi, pw, mm[k]);
      if (k & 1) pw *= s2;
    }
  }
  // The item's four N-terms from its record R, summed over the sixteen lanes
  // (on every lane); applied in FP64.
  __device__ __forceinline__ double total(const double* R, int m) const {
    constexpr int nT = RecLayout<MIXED>::nT;
    double acc[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int k = 0; k <= DT; ++k) {
        const double tr = R[kCheb + 2 * h * nT + k], ti = R[kCheb + (2 * h + 1) * nT + k];
        const double r = mr[k], q = mm[k];
        acc[2 * h] = fma(tr, r, k ? fma(ti, q, acc[2 * h]) : ti * q);
        acc[2 * h + 1] = fma(tr, q, k ? fma(-ti, r, acc[2 * h + 1]) : -ti * r);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = row_sum(acc[i]);
    const double lo = (m & 1) ? acc[1] : acc[0], hi = (m & 1) ? acc[3] : acc[2];
    return (m & 2) ? hi : lo;            // lane m of the row holds term m & 3
  }
};

// R(s) of a record's coefficients
__device__ __forceinline__ double phase_poly(const double* cR, double s) {
  const double s2 = s * s, s4 = s2 * s2;
  return estrin9(cR, s, s2, s4, s4 * s4);
}

// Whole blocks of the block-loop items: sixteen lanes per item, one per node;
// four items per wavefront, each lane looping over its item's blocks, two rows
// of the spectra in flight.  Items come in tile order and each XCD (block
// index mod 8) takes one contiguous eighth of them, so that the rows that many
// particles share at a time stay in its L2.  Bound by FP64 issue (about 75 vector
// operations per row and lane, 30 of them the phase and the row's choice, 20 the
// sine) at the three waves per SIMD that its registers allow.  A wave-uniform trip
// count, roundings by addition and DPP moves without an old value took 26 of 175
// operations per pair of rows, real and imaginary parts side by side one of two loads:
// 3.57e9 bins in 1.07 M items FP64 1.31 -> 1.16 ms, partial blocks 0.53 -> 0.49 ms.
template <bool MIXED>
__global__ __launch_bounds__(256, MIXED ? 4 : 3) void k_eval_blocks(
    Spectra<typename std::conditional<MIXED, float, double>::type> sp,
    const int32_t* __restrict__ list, const int32_t* __restrict__ nlist,
    const double* __restrict__ rec, double* __restrict__ partials) {
  typedef typename std::conditional<MIXED, float, double>::type DT_;
  typedef typename std::conditional<MIXED, float2, double2>::type DT2;
  typedef RecLayout<MIXED> L;
  __shared__ double2 s_tab[MIXED ? 1 : kSinTab];
  __shared__ double s_rec[4][4][kRecPad];
  if constexpr (!MIXED) {
    for (int k = threadIdx.x; k < kSinTab; k += blockDim.x) s_tab[k] = c_sincos[k];
    __syncthreads();
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int grp = lane >> 4, m = lane & 15;
  const int n = nlist[0];
  const int per = ((n + 7) / 8 + 15) & ~15;                 // items per XCD
  const int lo = min(n, (int)(blockIdx.x & 7) * per), hi = min(n, lo + per);
  const int step = (int)(gridDim.x >> 3) * 16;
  const double c = 0.5 * (double)(sp.L - 1);                // block centre
  double xs, xc;
  sincospi(((double)m + 0.5) / (double)kSpecNodes, &xs, &xc);
  const double y = c * xc;                                  // this lane's node
  sincospi(0.5 / (double)kSpecNodes, &xs, &xc);
  const double chord = 0.5 / (c * xc);                      // 1 / (distance of the end nodes)
  const double invQ = 1.0 / (double)sp.Q, slmax = (double)(sp.nslots - 1) * invQ;
  const int lg = __builtin_ctz(sp.L);
  int first = lo + (int)(blockIdx.x >> 3) * 16 + wv * 4;    // of this wave's four items
  for (; first < hi; first += step) {
    const int w = first + grp < hi ? list[first + grp] : -1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int wi = __builtin_amdgcn_readlane(w, 16 * i);
      if (wi >= 0 && lane < kRec) s_rec[wv][i][lane] = rec[(int64_t)wi * kRec + lane];
    }
    __builtin_amdgcn_wave_barrier();
    const double* R = s_rec[wv][grp];
    const double A = R[L::tail], Bp = R[L::tail + 1], B = R[L::tail + 2];
    const int flags = rec_int(R[L::tail + 3], 0), b0 = rec_int(R[L::tail + 3], 1);
    const int nb = rec_int(R[L::tail + 4], 0);
    const double alpha = R[L::tail + 5];
    const int degT = (flags >> 8) & 255, ch = flags >> 16;
    const int fb = (b0 + sp.L - 1) >> lg;                   // whole blocks [fb, fb + nrow)
    const int nrow = w >= 0 ? max(min((b0 + nb) >> lg, sp.nblk) - fb, 0) : 0;
    const double Ac = A + (B * c - rint(B * c));            // the slope's phase at a block's centre
    const int rows = row_max(nrow);
    const DT2* base = reinterpret_cast<const DT2*>(sp.S) +
                      ((int64_t)ch * sp.nblk + fb) * sp.nslots * kSpecNodes + m;
    auto loop = [&](auto dt) {
      Moments<MIXED, decltype(dt)::value> M;
      M.clear();
      const double row0 = (double)((fb << lg) - b0);
      for (int i0 = 0; i0 < rows; i0 += kBlkAhead) {
        double s[kBlkAhead], ph[kBlkAhead];
        const double mb0 = fma((double)i0, (double)sp.L, row0);
        DT_ a[kBlkAhead], b[kBlkAhead];
#pragma unroll
        for (int u = 0; u < kBlkAhead; ++u) {
          const int i = i0 + u;
          const double mb = mb0 + (double)(u * sp.L);
          s[u] = fma(alpha, mb + (c + y), -1.0);
          const double r = phase_poly(R, s[u]);   // R's head: its coefficients
          // the chord of the block's phase chooses the slope slot
          const double sl = fma(row_bcast<0>(r) - row_bcast<15>(r), chord, B);
          int q;
          const double qd = round_int(fmin(fmax(sl, 0.0), slmax), (double)sp.Q, q);
          ph[u] = (r + Ac) + fma(Bp, mb, fma(-invQ, qd, B) * y);
          a[u] = b[u] = DT_(0);
          if (i < nrow) {
            const DT2 v = base[((int64_t)i * sp.nslots + q) * kSpecNodes];
            a[u] = v.x;
            b[u] = v.y;
          }
        }
#pragma unroll
        for (int u = 0; u < kBlkAhead; ++u) M.add(ph[u], s[u], a[u], b[u], s_tab);
      }
      const double t = M.total(R, m);
      if (nrow > 0 && m < 4) partials[(int64_t)w * 8 + m] = t;
    };
    if constexpr (MIXED) {
      if (__any(nrow > 0 && degT > kDegTLow)) loop(std::integral_constant<int, kDegT>{});
      else loop(std::integral_constant<int, kDegTLow>{});
    } else {
      if (__any(nrow > 0 && degT > 7)) loop(std::integral_constant<int, 9>{});
      else if (__any(nrow > 0 && degT > 5)) loop(std::integral_constant<int, 7>{});
      else loop(std::integral_constant<int, 5>{});
    }
    __builtin_amdgcn_wave_barrier();     // the slots are rewritten for the next items
  }
}

// Partial blocks of the block-loop items, bin by bin.  With tiles of whole
// blocks only a partition's first and last item of a channel have any: sixteen
// lanes take the first item of a (partition, channel) or, in the second half
// of the groups, the last one where that is another, and add to the sums of
// its whole blocks.
template <bool MIXED>
__global__ __launch_bounds__(256, MIXED ? 4 : 3) void k_eval_edges(
    Grid g, int32_t Lb, int32_t nblk, int64_t ngroups, const int32_t* __restrict__ cnt,
    const int32_t* __restrict__ off, const uint8_t* __restrict__ xflag,
    const typename std::conditional<MIXED, float, double>::type* __restrict__ wr,
    const typename std::conditional<MIXED, float, double>::type* __restrict__ wi,
    const double* __restrict__ rec, double* __restrict__ partials) {
  typedef typename std::conditional<MIXED, float, double>::type DT_;
  typedef RecLayout<MIXED> L;
  __shared__ double2 s_tab[MIXED ? 1 : kSinTab];
  __shared__ double s_rec[4][4][kRecPad];
  if constexpr (!MIXED) {
    for (int k = threadIdx.x; k < kSinTab; k += blockDim.x) s_tab[k] = c_sincos[k];
    __syncthreads();
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int grp = lane >> 4, m = lane & 15;
  const int lg = __builtin_ctz(Lb);
  const int nch = g.chan.n;
  const int64_t step = (int64_t)gridDim.x * 16;
  for (int64_t first = (int64_t)blockIdx.x * 16 + wv * 4; first < 2 * ngroups; first += step) {
    const int64_t id = first + grp;
    int w = -1;
    if (id < 2 * ngroups) {
      const bool side = id >= ngroups;
      const int64_t pq = side ? id - ngroups : id, q = pq / nch;
      const int n = cnt[q];
      if (n > (side ? nch : 0)) {
        w = off[q] + (int)(pq - q * nch) + (side ? n - nch : 0);
        if (xflag[w] != kItemBlocks) w = -1;
      }
    }
    if (!__any(w >= 0)) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int wi_ = __builtin_amdgcn_readlane(w, 16 * i);
      if (wi_ >= 0 && lane < kRec) s_rec[wv][i][lane] = rec[(int64_t)wi_ * kRec + lane];
    }
    __builtin_amdgcn_wave_barrier();
    const double* R = s_rec[wv][grp];
    const double A = R[L::tail], Bp = R[L::tail + 1], alpha = R[L::tail + 5];
    const double kB = R[L::tail + 6];
    const int flags = rec_int(R[L::tail + 3], 0), b0 = rec_int(R[L::tail + 3], 1);
    const int nb = rec_int(R[L::tail + 4], 0);
    const int degT = (flags >> 8) & 255, ch = flags >> 16;
    const int b1 = b0 + nb;
    const int fb = (b0 + Lb - 1) >> lg, lb = min(b1 >> lg, nblk);
    const int h1 = min(fb << lg, b1), t0 = max(lb << lg, h1);   // bins [b0, h1) and [t0, b1)
    const int nh = (h1 - b0 + 15) >> 4;
    const int nrow = w >= 0 ? nh + ((b1 - t0 + 15) >> 4) : 0;
    const DT_* cwr = wr + (int64_t)ch * g.nbins;
    const DT_* cwi = wi + (int64_t)ch * g.nbins;
    const int rows = row_max(nrow);
    auto loop = [&](auto dt) {
      Moments<MIXED, decltype(dt)::value> M;
      M.clear();
      for (int i0 = 0; i0 < rows; i0 += kBlkAhead) {
        int j[kBlkAhead];
        DT_ a[kBlkAhead], b[kBlkAhead];
#pragma unroll
        for (int u = 0; u < kBlkAhead; ++u) {
          const int i = i0 + u;
          const bool head = i < nh;
          j[u] = (head ? b0 + 16 * i : t0 + 16 * (i - nh)) + m;
          a[u] = b[u] = DT_(0);
          if (i < nrow && j[u] < (head ? h1 : b1)) { a[u] = cwr[j[u]]; b[u] = cwi[j[u]]; }
        }
#pragma unroll
        for (int u = 0; u < kBlkAhead; ++u) {
          const double mi = (double)(j[u] - b0);
          const double s = fma(alpha, mi, -1.0);
          double ph = fma(Bp, mi, phase_poly(R, s)) + A;
          if constexpr (!MIXED) {
            const double jd = (double)(g.k_lo + j[u]);      // grid rounding, as in k_eval_interp
            ph = fma(kB, fma(jd, g.df, -(jd * g.df)), ph);
          }
          M.add(ph, s, a[u], b[u], s_tab);
        }
      }
      const double t = M.total(R, m);
      if (nrow > 0 && m < 4) {
        double* o = partials + (int64_t)w * 8 + m;
        *o = lb > fb ? *o + t : t;
      }
    };
    if (__any(nrow > 0)) {
      if constexpr (MIXED) {
        if (__any(nrow > 0 && degT > kDegTLow)) loop(std::integral_constant<int, kDegT>{});
        else loop(std::integral_constant<int, kDegTLow>{});
      } else {
        if (__any(nrow > 0 && degT > 7)) loop(std::integral_constant<int, 9>{});
        else if (__any(nrow > 0 && degT > 5)) loop(std::integral_constant<int, 7>{});
        else loop(std::integral_constant<int, 5>{});
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Refinement of the FP64 interpolating loop's partitions.  With beta =
// H^{-1} z the maximiser and r the data minus its projection on the template
// span, a template error dA and an error dH_q of the quadrature M-terms move
// F = 1/2 z^H H^{-1} z (Sec. II.A, Eq. coherent_F_stat) to first order by
//     dF = Re <r, dA beta> + Re <A beta, dA beta> - 1/2 beta^H dH_q beta
// (the last two vanish where the M-terms are summed from the same
// interpolated templates).  |A beta|^2 = 2F; for Gaussian noise <r, v> is a
// normal variable of variance at most |v|^2; an item whose transfer and phase
// interpolants are off by at most e relative to its largest transfer
// component m contributes at most 2 e^2 m^2 sum(u) to |dA_k|^2 (k = +, x),
// and each entry of its quadrature M-terms is off by at most g (the
// quadrature's end-point error times max u|T|^2 times its bin count).  So
//   |dF| <~ sqrt 2 (kappa + sqrt(2F)) b sqrt(sum (e m)^2 sum u) + b^2 sum g / 2
// with b = |beta_+| + |beta_x| and kappa = kRefineKappa covering six standard
// deviations of the noise and an unmatched signal of SNR 10 in the
// partition.  Where this exceeds budget * max(|F|, 1), the items whose share
// of either term is above half the budget's share are evaluated again
// exactly, which brings the remainder under the budget.  Partitions within a
// factor kFragile of the pseudo-inverse cut are refined whole (a small error
// could flip the rank decision).
//
// The block loop adds an error of its own to the items it takes: the sixteen-point
// interpolation, at most kSpecErrFp64 per sample, and the grid rounding, which the
// spectra take at the slot's slope, up to 2 pi |B - beta_q| e_j / df radians per bin,
// |B - beta_q| <= 1 / (2 Q), |e_j| half an ulp of f (spectra.hip).  Both multiply the
// template's two polarisations by one factor 1 + eps_j (to the change of T over a
// block), so that dA beta = eps A beta whatever beta is: |dA beta| <= max|eps| sqrt(2F)
// without the conditioning that b carries, and the partition's share is
//   (kappa + sqrt(2F)) sqrt(2F) max|eps|,
// at most kSpecGain max|eps| of max(F, 1) (at F = 1).  spec_fmax keeps that within half
// the budget; the terms above have the rest.  (At 2.5 years and Q = 512 it is
// 1.4e-11..8.7e-11 from 10 to 100 mHz.  Summed into e instead, with b's conditioning, it
// would send nearly every item of a 4096 x 64 batch to the exact loop: 2.8 -> 32.7 ms.)
constexpr double kRefineKappa = 16.0;
constexpr double kFragile = 1e3;
constexpr double kSpecErrFp64 = 1.6e-13;   // slope pi / 4, curvature 0.25 rad: 1.5e-13
constexpr double kSpecGain = 24.63;        // (kappa + sqrt 2) sqrt 2

// 2 pi |B - beta_q| / df at its largest, 0 where every k df is a double (df has `bits`
// significant bits, k at most 53 - bits)
static double spec_grid(const Grid& g, int32_t Q) {
  int e = 0, bits = 0;
  uint64_t m = (uint64_t)std::ldexp(std::frexp(g.df, &e), 53);
  while (!(m & 1)) m >>= 1;
  for (; m; m >>= 1) ++bits;
  return ((uint64_t)(g.k_lo + g.nbins - 1) >> (53 - bits)) == 0 ? 0.0 : kPi / (Q * g.df);
}

// The frequency (a power of two: half an ulp of f changes there) up to which the FP64
// block loop's error stays within half the refinement budget; items that reach above
// take the per-bin loop, which has each bin's rounding exactly.  Budget 5e-10 at 2.5
// years: 62.5 mHz with Q = 128, 125 mHz with Q = 256, 250 mHz with Q = 512.
double spec_fmax(const Grid& g, int32_t Q, double budget) {
  if (!(budget > 0.0)) return HUGE_VAL;                   // no estimate asked for
  const double eps = 0.5 * budget / kSpecGain - kSpecErrFp64, gr = spec_grid(g, Q);
  if (!(eps > 0.0)) return 0.0;
  return gr > 0.0 ? std::ldexp(1.0, std::ilogb(eps / gr) + 54) : HUGE_VAL;
}

// Sums of a partition's items [o, o + c): eight lanes, lane k the k-th of the
// eight terms (an item's partials are one 64-byte line), Neumaier sums in item
// order.  On return every lane of the group holds all eight.  One thread per
// partition, reading eight values 64 bytes apart per item, took 580 us (k_mark)
// and 196 us (k_solve) for 6144 coherent particles of ~360 items each.
__device__ __forceinline__ void partition_sums(const double* __restrict__ partials, int o, int c,
                                               int k, double a[8]) {
  double s = 0.0, e = 0.0;
  const double* x0 = partials + (int64_t)o * 8 + k;
  auto add = [&](double x) {
    const double t = s + x;
    e += (fabs(s) >= fabs(x)) ? (s - t) + x : (x - t) + s;
    s = t;
  };
  // sixteen loads under way at a time, the additions in the items' order: a partition
  // of 160 items (one whole-band particle) waits ten times instead of forty, k_mark
  // 23 -> 13 us and k_solve 10 -> 8; partitions of a few items are not affected
  int i = 0;
  for (; i + 16 <= c; i += 16) {
    double x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = x0[(int64_t)(i + u) * 8];
#pragma unroll
    for (int u = 0; u < 16; ++u) add(x[u]);
  }
#pragma unroll 4
  for (; i < c; ++i) add(x0[(int64_t)i * 8]);
  s += e;
#pragma unroll
  for (int j = 0; j < 8; ++j) a[j] = __shfl(s, j, 8);
}

// Eight lanes per partition.
__global__ __launch_bounds__(256) void k_mark(Grid g, double grid_term,
                                              const PartConst* __restrict__ pc, int64_t n,
                                              const int32_t* __restrict__ bounds,
                                              int32_t stride, const int32_t* __restrict__ cnt,
                                              const int32_t* __restrict__ off,
                                              const double* __restrict__ partials,
                                              const uint8_t* __restrict__ xflag,
                                              const float2* __restrict__ xerr, double budget,
                                              int32_t* __restrict__ refine,
                                              int32_t* __restrict__ nrefine) {
  const int64_t q = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 3;
  const int k = threadIdx.x & 7, lane = threadIdx.x & 63;
  int o = 0, c = 0, last = 0;                  // no items: the group only takes part in the scan
  if (q < n * stride) {
    const int64_t p = q / stride;
    const PartConst& P = pc[p];
    const int l = (int)(q - p * stride);
    if (l < P.np && P.status == kStatusOk) {
      o = off[q];
      c = cnt[q];
      last = bounds[p * (stride + 1) + l + 1];
    }
  }
  // the items' error terms, every eighth item per lane
  int ninterp = 0, nblocks = 0;
  double s2 = 0.0, mt = 0.0;
  for (int i = k; i < c; i += 32) {              // four of them under way
    uint8_t f[4];
    float2 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int at = o + min(i + 8 * u, c - 1);
      f[u] = xflag[at];
      x[u] = xerr[at];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + 8 * u < c && f[u] != kItemExact) {
        ++ninterp;
        nblocks += f[u] == kItemBlocks ? 1 : 0;
        s2 = fma((double)x[u].x, (double)x[u].x, s2);
        mt += (double)x[u].y;
      }
  }
#pragma unroll
  for (int d = 4; d > 0; d >>= 1) {
    ninterp += __shfl_xor(ninterp, d, 8);
    nblocks += __shfl_xor(nblocks, d, 8);
    s2 += __shfl_xor(s2, d, 8);
    mt += __shfl_xor(mt, d, 8);
  }
  double a[8];
  partition_sums(partials, o, ninterp > 0 ? c : 0, k, a);
  const double Pm = a[4], Qm = a[5], rr = a[6], ri = a[7];
  const double hs = 0.5 * (Pm + Qm), hd = 0.5 * (Pm - Qm);
  const double lp = hs + sqrt(hd * hd + rr * rr + ri * ri);
  const double lm = (Pm * Qm - (rr * rr + ri * ri)) / lp;
  const bool all = !(lp > 0.0) || !(lm > kFragile * kRankCut * lp);
  double thr_t = 0.0, thr_m = 0.0;
  bool some = ninterp > 0;
  if (some && !all) {
    double beta[4];
    solve_beta(a, beta);
    const double F = solve_partition(a);
    const double b = hypot(beta[0], beta[1]) + hypot(beta[2], beta[3]);
    const double kt = 1.4142135623730951 * (kRefineKappa + sqrt(2.0 * fmax(F, 0.0))) * b;
    const double km = 0.5 * b * b;
    double tol = budget * fmax(fabs(F), 1.0);
    if (nblocks > 0) {
      const double f = (double)(g.k_lo + last) * g.df, rF = sqrt(2.0 * fmax(F, 0.0));
      const double eps = fma(grid_term, ldexp(1.0, __builtin_amdgcn_frexp_exp(f) - 54), kSpecErrFp64);
      tol = fmax(tol - (kRefineKappa + rF) * rF * eps, 0.5 * tol);
    }
    some = !(kt * sqrt(s2) + km * mt <= tol);
    // refining every item above these leaves at most tol / 2 in each term
    thr_t = 0.5 * tol / (kt * sqrt((double)ninterp));
    thr_m = 0.5 * tol / (km * (double)ninterp);
  }
  if (!__any(some)) return;
  auto sel = [&](int i) {
    if (xflag[o + i] == kItemExact) return false;
    const float2 x = xerr[o + i];
    return all || (double)x.x > thr_t || (double)x.y > thr_m;
  };
  int ns = 0;
  for (int i = some ? k : c; i < c; i += 8) ns += sel(i) ? 1 : 0;
  // one place in the list for the wavefront's items (an atomic per item took
  // 0.9 ms for 421,783 of them)
  int at = ns;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(at, d, 64);
    if (lane >= d) at += y;
  }
  const int tot = __shfl(at, 63, 64);
  if (tot == 0) return;
  int base = 0;
  if (lane == 0) base = atomicAdd(nrefine, tot);
  at += __shfl(base, 0, 64) - ns;
  for (int i = some ? k : c; i < c; i += 8)
    if (sel(i)) refine[at++] = o + i;
}

// Bins of the last evaluation's items by the kind of per-bin work the
// interpolating loop did on them: out[0..2] direct phase and sine per bin at
// transfer degree 5, 7, 9, out[3..5] the difference recurrence at degree 5, 7,
// 9 (mixed path: [0] degree 4 and [2] degree 6 with all nine phase
// differences, [3] and [5] the same with four), out[6] evaluated exactly
// (rejects; refined items count where the interpolating loop ran them).
// out[7 + k] (k < 6): the lanes with bins (runs) of the items of kind k, each
// of which does its kind's per-lane work once (recurrence set-up, moments to
// power form, coefficients); out[13]: items evaluated exactly.
template <bool MIXED>
__global__ __launch_bounds__(256) void k_bin_mix(const int2* __restrict__ items,
                                                 const int32_t* __restrict__ total,
                                                 const int32_t* __restrict__ bounds,
                                                 int32_t stride, Tiling tl, int32_t nch,
                                                 const double* __restrict__ rec,
                                                 const uint8_t* __restrict__ xflag,
                                                 unsigned long long* __restrict__ out) {
  typedef RecLayout<MIXED> L;
  __shared__ unsigned long long acc[kBinMix];
  if (threadIdx.x < kBinMix) acc[threadIdx.x] = 0ull;
  __syncthreads();
  const int W = total[0];
  for (int w = blockIdx.x * blockDim.x + threadIdx.x; w < W; w += gridDim.x * blockDim.x) {
    const int2 it = items[w];
    const int p = it.x / stride, l = it.x - p * stride;
    const int32_t* bp = bounds + (int64_t)p * (stride + 1);
    int b0, b1;
    item_bins(bp[l], bp[l + 1], it.y, item_chan(it.y, tl, nch), tl, b0, b1);
    const int nb = b1 - b0;
    int kind = 6, runs = 1;
    if (xflag[w] != kItemExact) {
      const double* r = rec + (int64_t)w * kRec;
      const int flags = rec_int(r[L::tail + 3], 0), state = flags & 255;
      const int deg = (flags >> 8) & 255;
      const bool dr = state != kRecBins;
      kind = (MIXED ? (deg == kDegTLow ? 0 : 2) : (deg == 5 ? 0 : (deg == 7 ? 1 : 2))) + (dr ? 3 : 0);
      // the recurrence's and the mixed loop's lanes take runs of Lr
      // contiguous bins, the FP64 direct form's lanes every 64th bin
      // (a block-loop item: its sixteen lanes)
      const int Lr = ((nb + 63) >> 6) | 1;
      runs = state == kRecBlocks ? kSpecNodes
                                 : ((MIXED || dr) ? (nb + Lr - 1) / Lr : min(nb, 64));
    }
    atomicAdd(&acc[kind], (unsigned long long)nb);
    atomicAdd(&acc[7 + kind], (unsigned long long)runs);
  }
  __syncthreads();
  if (threadIdx.x < kBinMix && acc[threadIdx.x]) atomicAdd(&out[threadIdx.x], acc[threadIdx.x]);
}

void launch_bin_mix(bool mixed, int32_t stride, const Tiling& tl, int32_t nch, const WorkSpace& ws,
                    unsigned long long* out, hipStream_t s) {
  hipLaunchKernelGGL(mixed ? k_bin_mix<true> : k_bin_mix<false>, dim3(1024), dim3(256), 0, s,
                     ws.items, ws.total, ws.bounds, stride, tl, nch, ws.rec, ws.xflag, out);
}

// ---- grouping of the work items by loop and bin tile -------------------------
__global__ void k_tile_zero(int32_t* __restrict__ tcnt, int32_t* __restrict__ tcur, int32_t n2,
                            int32_t* __restrict__ tile_ctr) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n2) { tcnt[i] = 0; tcur[i] = 0; }
  if (i == 0) tile_ctr[0] = 0;
}

// Where item w is counted: its tile, of the block loop or (+ ntiles) of the
// per-bin loop; -1: the exact loop takes it.
__device__ __forceinline__ int tile_key(const int2* __restrict__ items,
                                        const uint8_t* __restrict__ xflag, int32_t ntiles, int w) {
  const uint8_t x = xflag[w];
  if (x == kItemExact) return -1;
  const int t = items[w].y >> 3;
  return x == kItemBlocks ? t : ntiles + t;
}

// Items per key.  When the keys fit in LDS the block first counts its own
// items there and then adds its non-zero counts to the global ones: with few
// tiles (a narrow band) every item would otherwise hit the same few counters
// (counting in the node kernel by global atomics cost 1.5 ms at 872,322 items
// on 198 tiles, and 0.2 ms at 2 million on 3468).  One large block per CU: a block clears
// and adds up all its counters (1.07 M items on 2774 tiles, both kernels: 63 us with
// 1024 blocks of 256, 47 with 512, 26 with 256 of 1024).
constexpr int kTileHist = 8192;

__global__ __launch_bounds__(1024) void k_tile_count(const int2* __restrict__ items,
                                                    const int32_t* __restrict__ total,
                                                    const uint8_t* __restrict__ xflag,
                                                    int32_t ntiles, int32_t* __restrict__ tcnt) {
  __shared__ int32_t h[kTileHist];
  const int nk = 2 * ntiles;
  const bool local = nk <= kTileHist;
  const int W = total[0];
  if (local) {
    for (int i = threadIdx.x; i < nk; i += blockDim.x) h[i] = 0;
    __syncthreads();
  }
  for (int w = blockIdx.x * blockDim.x + threadIdx.x; w < W; w += gridDim.x * blockDim.x) {
    const int t = tile_key(items, xflag, ntiles, w);
    if (t < 0) continue;
    if (local) atomicAdd(&h[t], 1);
    else atomicAdd(&tcnt[t], 1);
  }
  if (local) {
    __syncthreads();
    for (int i = threadIdx.x; i < nk; i += blockDim.x)
      if (h[i]) atomicAdd(&tcnt[i], h[i]);
  }
}

// Exclusive scans of the per-tile item counts into off[0..2 n] (the block
// loop's tiles, then the per-bin loop's) and of the per-bin loop's unit counts
// ceil(cnt / kUnitItems) into uoff[0..n] (a unit is its scheduling step: one
// tile, up to kUnitItems of its items).  One block.
__global__ __launch_bounds__(1024) void k_tile_scan(const int32_t* __restrict__ tcnt, int32_t n,
                                                    int32_t* __restrict__ off,
                                                    int32_t* __restrict__ uoff) {
  __shared__ int32_t sh[1024];
  const int t = threadIdx.x;
  const int per = (2 * n + 1023) / 1024;
  const int a = min(2 * n, t * per), b = min(2 * n, a + per);
  int32_t sum = 0, usum = 0, tot, utot;
  for (int i = a; i < b; ++i) {
    sum += tcnt[i];
    if (i >= n) usum += (tcnt[i] + kUnitItems - 1) / kUnitItems;
  }
  int32_t run = block_excl_scan(sum, sh, tot);
  int32_t urun = block_excl_scan(usum, sh, utot);
  if (t == 0) {
    off[2 * n] = tot;
    uoff[n] = utot;
  }
  for (int i = a; i < b; ++i) {
    off[i] = run;
    run += tcnt[i];
    if (i >= n) {
      uoff[i - n] = urun;
      urun += (tcnt[i] + kUnitItems - 1) / kUnitItems;
    }
  }
}

// Interpolated items into (loop, tile) order.  With the keys in LDS, the block
// ranks its items per key locally and reserves one range per key with a single
// global atomic.
__global__ __launch_bounds__(1024) void k_tile_scatter(const int2* __restrict__ items,
                                                      const int32_t* __restrict__ total,
                                                      const uint8_t* __restrict__ xflag,
                                                      int32_t ntiles,
                                                      const int32_t* __restrict__ off,
                                                      int32_t* __restrict__ tcur,
                                                      int32_t* __restrict__ tile_items) {
  __shared__ int32_t h[kTileHist];
  const int nk = 2 * ntiles;
  const bool local = nk <= kTileHist;
  const int W = total[0];
  if (!local) {
    for (int w = blockIdx.x * blockDim.x + threadIdx.x; w < W; w += gridDim.x * blockDim.x) {
      const int t = tile_key(items, xflag, ntiles, w);
      if (t >= 0) tile_items[off[t] + atomicAdd(&tcur[t], 1)] = w;
    }
    return;
  }
  for (int i = threadIdx.x; i < nk; i += blockDim.x) h[i] = 0;
  __syncthreads();
  for (int w = blockIdx.x * blockDim.x + threadIdx.x; w < W; w += gridDim.x * blockDim.x) {
    const int t = tile_key(items, xflag, ntiles, w);
    if (t >= 0) atomicAdd(&h[t], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nk; i += blockDim.x)    // counts -> reserved bases
    if (h[i]) h[i] = off[i] + atomicAdd(&tcur[i], h[i]);
  __syncthreads();
  for (int w = blockIdx.x * blockDim.x + threadIdx.x; w < W; w += gridDim.x * blockDim.x) {
    const int t = tile_key(items, xflag, ntiles, w);
    if (t >= 0) tile_items[atomicAdd(&h[t], 1)] = w;
  }
}

// Count, scan and scatter in one block, for few items (host bound kGroupOnce)
// on few tiles: one launch instead of three.
constexpr int64_t kGroupOnce = 32768;

__global__ __launch_bounds__(1024) void k_tile_group(const int2* __restrict__ items,
                                                     const int32_t* __restrict__ total,
                                                     const uint8_t* __restrict__ xflag,
                                                     int32_t ntiles, int32_t* __restrict__ off,
                                                     int32_t* __restrict__ uoff,
                                                     int32_t* __restrict__ tile_items) {
  __shared__ int32_t h[kTileHist];
  __shared__ int32_t sh[1024];
  const int t = threadIdx.x, nk = 2 * ntiles;
  const int W = total[0];
  for (int i = t; i < nk; i += 1024) h[i] = 0;
  __syncthreads();
  for (int w = t; w < W; w += 1024) {
    const int k = tile_key(items, xflag, ntiles, w);
    if (k >= 0) atomicAdd(&h[k], 1);
  }
  __syncthreads();
  const int per = (nk + 1023) / 1024, a = min(nk, t * per), b = min(nk, a + per);
  int32_t sum = 0, usum = 0, tot, utot;
  for (int i = a; i < b; ++i) {
    sum += h[i];
    if (i >= ntiles) usum += (h[i] + kUnitItems - 1) / kUnitItems;
  }
  int32_t run = block_excl_scan(sum, sh, tot);
  int32_t urun = block_excl_scan(usum, sh, utot);
  if (t == 0) {
    off[nk] = tot;
    uoff[ntiles] = utot;
  }
  for (int i = a; i < b; ++i) {
    const int32_t c = h[i];
    off[i] = run;
    h[i] = run;
    run += c;
    if (i >= ntiles) {
      uoff[i - ntiles] = urun;
      urun += (c + kUnitItems - 1) / kUnitItems;
    }
  }
  __syncthreads();
  for (int w = t; w < W; w += 1024) {
    const int k = tile_key(items, xflag, ntiles, w);
    if (k >= 0) tile_items[atomicAdd(&h[k], 1)] = w;
  }
}

// every item is evaluated exactly: the reject count equals the item count
__global__ void k_copy_count(const int32_t* __restrict__ total, int32_t* __restrict__ ndirect) {
  if (threadIdx.x == 0) ndirect[0] = total[0];
}

// Chebyshev tables (long double on the host): node s_k = cos(pi (k + 1/2) / K);
// interpolant coefficients c_j = (2 / K) sum_k v_k cos(pi j (k + 1/2) / K)
// (c_0 halved) of p = sum_j c_j T_j(s); T_j expanded in monomials by
// T_{j+1} = 2 s T_j - T_{j-1}.
static double* g_ssum[64] = {};   // per device: S_j(nb) table (lives until the process ends)

int interp_tables_init() {
  static bool done[64] = {false};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -1;
  if (dev >= 0 && dev < 64 && done[dev]) return 0;
  if (spectra_tables_init() != 0) return -1;
  const int K = kCheb;
  const long double pi = 3.141592653589793238462643383279502884L;
  long double M[kCheb][kCheb] = {};
  M[0][0] = 1.0L;
  M[1][1] = 1.0L;
  for (int j = 1; j + 1 < K; ++j)
    for (int n = 0; n < K; ++n)
      M[j + 1][n] = (n > 0 ? 2.0L * M[j][n - 1] : 0.0L) - M[j - 1][n];
  double S[kCheb], G[kCheb][kCheb], E[2][kCheb], G6[kCheb][kDegT + 1], E6[2][kCheb];
  for (int kk = 0; kk < K; ++kk) {
    S[kk] = (double)cosl(pi * (kk + 0.5L) / K);
    long double lm = 0.0L, lp = 0.0L, lm6 = 0.0L, lp6 = 0.0L;
    for (int n = 0; n < K; ++n) {
      long double gsum = 0.0L, g6 = 0.0L;
      for (int j = 0; j < K; ++j) {
        long double cj = (2.0L / K) * cosl(pi * j * (kk + 0.5L) / K) * (j == 0 ? 0.5L : 1.0L);
        gsum += cj * M[j][n];
        if (j <= kDegT) g6 += cj * M[j][n];
      }
      G[kk][n] = (double)gsum;
      lp += gsum;
      lm += (n & 1) ? -gsum : gsum;
      if (n <= kDegT) {
        G6[kk][n] = (double)g6;
        lp6 += g6;
        lm6 += (n & 1) ? -g6 : g6;
      }
    }
    E[0][kk] = (double)lm;
    E[1][kk] = (double)lp;
    E6[0][kk] = (double)lm6;
    E6[1][kk] = (double)lp6;
  }
  if (hipMemcpyToSymbol(HIP_SYMBOL(c_cheb_s), S, sizeof(S)) != hipSuccess) return -1;
  double R9[kCheb][kLanesItem], R6[kCheb][kLanesItem];
  for (int kk = 0; kk < K; ++kk) {
    for (int n = 0; n < K; ++n) {
      R9[kk][n] = G[kk][n];
      R6[kk][n] = n <= kDegT ? G6[kk][n] : 0.0;
    }
    for (int e = 0; e < 2; ++e) {
      R9[kk][kCheb + e] = E[e][kk];
      R6[kk][kCheb + e] = E6[e][kk];
    }
  }
  if (hipMemcpyToSymbol(HIP_SYMBOL(c_row9), R9, sizeof(R9)) != hipSuccess) return -1;
  {
    double2 tab[kSinTab];
    for (int i = 0; i < kSinTab; ++i) {
      const long double a = 2.0L * pi * (long double)i / (long double)kSinTab;
      tab[i] = make_double2((double)sinl(a), (double)cosl(a));
    }
    if (hipMemcpyToSymbol(HIP_SYMBOL(c_sincos), tab, sizeof(tab)) != hipSuccess) return -1;
  }
  {
    double2 tab[kLogTab];
    for (int i = 0; i < kLogTab; ++i) {
      const double y0 = rint((double)ldexpl(logl(1.0L + (i + 0.5L) / kLogTab), 40));
      long double best = 1.0L;
      for (int j = -64; j <= 64; ++j) {      // log c near the interval's middle, best 1 / c
        const double y = ldexp(y0 + j, -40);
        const long double rc = expl(-(long double)y), e = fabsl(rc - (long double)(double)rc);
        if (e < best) {
          best = e;
          tab[i] = make_double2((double)rc, y);
        }
      }
    }
    if (hipMemcpyToSymbol(HIP_SYMBOL(c_logtab), tab, sizeof(tab)) != hipSuccess) return -1;
  }
  if (hipMemcpyToSymbol(HIP_SYMBOL(c_row6), R6, sizeof(R6)) != hipSuccess) return -1;
  // truncations after degree 5 and 7 (FP64 loop)
  double Gt[2][kCheb][kCheb], Et[2][2][kCheb];
  for (int v = 0; v < 2; ++v) {
    const int dmax = v == 0 ? 5 : 7;
    for (int kk = 0; kk < K; ++kk) {
      long double lm = 0.0L, lp = 0.0L;
      for (int n = 0; n < K; ++n) {
        long double gsum = 0.0L;
        for (int j = 0; j <= dmax; ++j)
          gsum += (2.0L / K) * cosl(pi * j * (kk + 0.5L) / K) * (j == 0 ? 0.5L : 1.0L) * M[j][n];
        Gt[v][kk][n] = (double)gsum;
        lp += gsum;
        lm += (n & 1) ? -gsum : gsum;
      }
      Et[v][0][kk] = (double)lm;
      Et[v][1][kk] = (double)lp;
    }
  }
  double Rt[2][kCheb][kLanesItem];
  for (int v = 0; v < 2; ++v)
    for (int kk = 0; kk < K; ++kk) {
      for (int n = 0; n < K; ++n) Rt[v][kk][n] = Gt[v][kk][n];
      for (int e = 0; e < 2; ++e) Rt[v][kk][kCheb + e] = Et[v][e][kk];
    }
  if (hipMemcpyToSymbol(HIP_SYMBOL(c_rowt), Rt, sizeof(Rt)) != hipSuccess) return -1;
  {
    // truncation after degree kDegTLow (mixed loop)
    double R4[kCheb][kLanesItem];
    for (int kk = 0; kk < K; ++kk) {
      long double lm = 0.0L, lp = 0.0L;
      for (int n = 0; n < K; ++n) {
        long double gsum = 0.0L;
        for (int j = 0; j <= kDegTLow; ++j)
          gsum += (2.0L / K) * cosl(pi * j * (kk + 0.5L) / K) * (j == 0 ? 0.5L : 1.0L) * M[j][n];
        R4[kk][n] = (double)gsum;
        lp += gsum;
        lm += (n & 1) ? -gsum : gsum;
      }
      R4[kk][kCheb] = (double)lm;
      R4[kk][kCheb + 1] = (double)lp;
    }
    if (hipMemcpyToSymbol(HIP_SYMBOL(c_row4), R4, sizeof(R4)) != hipSuccess) return -1;
  }
  // quadrature weights' Chebyshev part (even degrees only)
  double D[5][kCheb];
  for (int i = 0; i < 5; ++i)
    for (int kk = 0; kk < K; ++kk)
      D[i][kk] = (double)((2.0L / K) * cosl(pi * (2 * i) * (kk + 0.5L) / K) * (i == 0 ? 0.5L : 1.0L));
  if (hipMemcpyToSymbol(HIP_SYMBOL(c_cheb_D), D, sizeof(D)) != hipSuccess) return -1;
  // inverse Gram matrix of the u-tile least-squares fit (Gauss-Jordan)
  long double Gm[kUCoef][2 * kUCoef] = {};
  for (int m = 0; m < kUTile; ++m) {
    const long double s = 2.0L * m / (kUTile - 1) - 1.0L;
    long double tv[kUCoef];
    tv[0] = 1.0L;
    tv[1] = s;
    for (int k = 2; k < kUCoef; ++k) tv[k] = 2.0L * s * tv[k - 1] - tv[k - 2];
    for (int a = 0; a < kUCoef; ++a)
      for (int b = 0; b < kUCoef; ++b) Gm[a][b] += tv[a] * tv[b];
  }
  for (int a = 0; a < kUCoef; ++a) Gm[a][kUCoef + a] = 1.0L;
  for (int c = 0; c < kUCoef; ++c) {
    int piv = c;
    for (int r = c + 1; r < kUCoef; ++r)
      if (fabsl(Gm[r][c]) > fabsl(Gm[piv][c])) piv = r;
    for (int b = 0; b < 2 * kUCoef; ++b) { long double x = Gm[c][b]; Gm[c][b] = Gm[piv][b]; Gm[piv][b] = x; }
    const long double d = Gm[c][c];
    for (int b = 0; b < 2 * kUCoef; ++b) Gm[c][b] /= d;
    for (int r = 0; r < kUCoef; ++r)
      if (r != c) {
        const long double f = Gm[r][c];
        for (int b = 0; b < 2 * kUCoef; ++b) Gm[r][b] -= f * Gm[c][b];
      }
  }
  double Gi[kUCoef][kUCoef];
  for (int a = 0; a < kUCoef; ++a)
    for (int b = 0; b < kUCoef; ++b) Gi[a][b] = (double)Gm[a][kUCoef + b];
  if (hipMemcpyToSymbol(HIP_SYMBOL(c_ufit_Ginv), Gi, sizeof(Gi)) != hipSuccess) return -1;
  // quadrature table S_j(nb), one per device
  double* tab = nullptr;
  if (hipMalloc((void**)&tab, sizeof(double) * 5 * (kSsumMax + 1)) != hipSuccess) return -1;
  hipLaunchKernelGGL(k_sincos_table, dim3(1), dim3(kSinTab), 0, 0);
  hipLaunchKernelGGL(k_cheb_sums, dim3((kSsumMax + 256) / 256), dim3(256), 0, 0, tab);
  if (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess) return -1;
  if (dev >= 0 && dev < 64) {
    g_ssum[dev] = tab;
    done[dev] = true;
  }
  return 0;
}

const double* cheb_sums_table() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  return g_ssum[dev];
}

// ---------------------------------------------------------------------------
// surrogate for the eccentric phase term (App. A): training data, knots,
// spot check against the analytic term, per-particle decision
// ---------------------------------------------------------------------------
// network inputs (f, Mc, e0) mapped to [-1, 1] over f in [10, 100] mHz,
// Mc in [10, 50] Msun, e0 in [0, 0.15]
__device__ __forceinline__ float nn_f(double f) { return (float)(2.0 * (f - 0.01) / 0.09 - 1.0); }

// Training samples from the plain template code: target y = te / (ecc_k tN),
// the eccentric term in units of e0^2 and the Newtonian phase.
__global__ void k_sur_data(uint64_t seed, int64_t n, float* __restrict__ X, float* __restrict__ T) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint64_t ctr[4] = {(uint64_t)i, 0ull, 0ull, 0ull}, o[4];
  philox4x64_10(ctr, seed, 0x5u, o);
  double u0 = (double)(o[0] >> 11) * 0x1.0p-53, u1 = (double)(o[1] >> 11) * 0x1.0p-53,
         u2 = (double)(o[2] >> 11) * 0x1.0p-53;
  double f = 0.01 + 0.09 * u0, mc = 10.0 + 40.0 * u1, e0 = 1e-4 + (0.15 - 1e-4) * u2;
  double th[6] = {0.0, mc, 0.0, 0.0, 0.0, e0};
  PartConst P;
  fill_constants(P, th);
  double tN, te;
  newton_and_ecc(P, f, tN, te);
  T[i] = (float)(te / (P.ecc_k * tN));
  X[3 * i + 0] = nn_f(f);
  X[3 * i + 1] = (float)P.nn_mc;
  X[3 * i + 2] = (float)P.nn_e0;
}

// four knots per partition (bins spread evenly over the partition), for
// particles with Np >= kSurMinNp; one thread per (partition, knot)
__device__ __forceinline__ bool sur_candidate(const PartConst& P, int l, const int32_t* bp) {
  return P.status == kStatusOk && P.np >= kSurMinNp && l < P.np && (bp[l + 1] - bp[l]) >= 4;
}
__device__ __forceinline__ int knot_bin(const int32_t* bp, int l, int a) {
  int nb = bp[l + 1] - bp[l];
  return bp[l] + (a * (nb - 1)) / 3;
}

__global__ void k_sur_knots(Grid g, const PartConst* __restrict__ pc,
                            const int32_t* __restrict__ bounds, int32_t stride, int64_t n,
                            int64_t rows, float* __restrict__ X) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= rows) return;
  if (t >= n * stride * 4) {   // padding rows of the network batch
    X[3 * t + 0] = 0.f; X[3 * t + 1] = 0.f; X[3 * t + 2] = 0.f;
    return;
  }
  int64_t q = t >> 2;
  int a = (int)(t & 3);
  int64_t p = q / stride;
  int l = (int)(q - p * stride);
  const PartConst& P = pc[p];
  const int32_t* bp = bounds + p * (stride + 1);
  float x0 = 0.f, x1 = 0.f, x2 = 0.f;
  if (sur_candidate(P, l, bp)) {
    x0 = nn_f(bin_freq(g, knot_bin(bp, l, a)));
    x1 = (float)P.nn_mc;
    x2 = (float)P.nn_e0;
  }
  X[3 * t + 0] = x0; X[3 * t + 1] = x1; X[3 * t + 2] = x2;
}

// knot values -> Lagrange coefficients; mismatch estimate from the residual of
// the interpolated surrogate against the analytic term at the four knots and
// the three mid-points, after removing its mean (a constant phase per
// partition is absorbed by the statistic): mm = (2 pi)^2 var(residual)
__global__ void k_sur_check(Grid g, const PartConst* __restrict__ pc,
                            const int32_t* __restrict__ bounds, int32_t stride, int64_t n,
                            const float* __restrict__ ynn, double* __restrict__ ek,
                            double* __restrict__ mm) {
  int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n * stride) return;
  int64_t p = q / stride;
  int l = (int)(q - p * stride);
  const PartConst& P = pc[p];
  const int32_t* bp = bounds + p * (stride + 1);
  if (!sur_candidate(P, l, bp)) {
    mm[q] = (P.status == kStatusOk && P.np >= kSurMinNp && l < P.np) ? 1e300 : 0.0;
    return;
  }
  double xa[4], va[4];
  for (int a = 0; a < 4; ++a) {
    xa[a] = bin_freq(g, knot_bin(bp, l, a));
    double tN, te;
    newton_and_ecc(P, xa[a], tN, te);
    va[a] = P.ecc_k * tN * (double)ynn[4 * q + a];
  }
  double* e = ek + 8 * q;
  for (int a = 0; a < 4; ++a) {
    double den = 1.0;
    for (int b = 0; b < 4; ++b)
      if (b != a) den *= xa[a] - xa[b];
    e[a] = xa[a];
    e[4 + a] = va[a] / den;
  }
  double r[7], mean = 0.0;
  for (int i = 0; i < 7; ++i) {
    int j = (i < 4) ? knot_bin(bp, l, i)
                    : (knot_bin(bp, l, i - 4) + knot_bin(bp, l, i - 3)) / 2;
    double f = bin_freq(g, j);
    double tN, te;
    newton_and_ecc(P, f, tN, te);
    r[i] = knot_interp(e, f) - te;
    mean += r[i];
  }
  mean /= 7.0;
  double var = 0.0;
  for (int i = 0; i < 7; ++i) var += (r[i] - mean) * (r[i] - mean);
  mm[q] = 4.0 * kPi * kPi * var / 7.0;
}

// particle uses the surrogate when every partition's estimate is <= thr
__global__ void k_sur_decide(PartConst* __restrict__ pc, int64_t n, int32_t stride,
                             const double* __restrict__ mm, double thr,
                             unsigned long long* __restrict__ counters) {
  int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  PartConst& P = pc[p];
  if (P.status != kStatusOk || P.np < kSurMinNp) return;
  double worst = 0.0;
  for (int l = 0; l < P.np; ++l) worst = fmax(worst, mm[p * stride + l]);
  int use = worst <= thr ? 1 : 0;
  P.sur = use;
  atomicAdd(counters + (use ? 0 : 1), 1ull);
}

// ---------------------------------------------------------------------------
// solve and mean
// ---------------------------------------------------------------------------
// Constant phase (turns) the statistic's template drops and the App. A
// waveform carries: -1/8 and the f-independent part of the alpha_5 term,
// c5' cN vfac^5 (1 + 3 ln sqrt 6).
__device__ __forceinline__ double dropped_phase(const PartConst& P) {
  double ph0 = -0.125 + P.c5v5 * (1.0 + 1.5 * log(6.0));
  return ph0 - rint(ph0);
}

// a_1..a_4 of the App. B basis from the pair beta solved against the scaled
// bin data (w, u) -> (gam w, gam^2 u): the template's beta is gam beta, the
// dropped phase turns it by e^{2 pi i ph0}, and s = (a1 - i a3) T+ g +
// (-a2 + i a4) Tx g.
__device__ __forceinline__ void amps_from_beta(const PartConst& P, const double* b, double gam,
                                               double* a) {
  double sc, cc;
  sincospi(2.0 * dropped_phase(P), &sc, &cc);
  const double pr = gam * (b[0] * cc - b[1] * sc), pi = gam * (b[1] * cc + b[0] * sc);
  const double xr = gam * (b[2] * cc - b[3] * sc), xi = gam * (b[3] * cc + b[2] * sc);
  a[0] = pr;
  a[1] = -xr;
  a[2] = -pi;
  a[3] = xi;
}

// One block per particle: eight lanes per partition (partition_sums), then the
// first wavefront takes the mean, lanes every 64th partition and a fixed
// butterfly (the result does not depend on the launch).
__global__ __launch_bounds__(1024) void k_solve(const PartConst* __restrict__ pc, int32_t stride,
                                               const int32_t* __restrict__ cnt,
                                               const int32_t* __restrict__ off,
                                               const double* __restrict__ partials,
                                               double* __restrict__ Fl,
                                               double* __restrict__ F_hat,
                                               double* __restrict__ F_part, int64_t part_stride,
                                               double* __restrict__ amps,
                                               const double* __restrict__ umax,
                                               unsigned long long* __restrict__ bin_counter) {
  const int64_t p = blockIdx.x;
  const PartConst& P = pc[p];
  const int k = threadIdx.x & 7;
  const int status = P.status, np = P.np;
  if (status == kStatusInvalid) {
    if (threadIdx.x == 0) F_hat[p] = __builtin_nan("");
    for (int l = threadIdx.x; l < np && l < part_stride; l += blockDim.x) {
      if (F_part) F_part[p * part_stride + l] = __builtin_nan("");
      if (amps)
        for (int i = 0; i < 4; ++i) amps[(p * part_stride + l) * 4 + i] = __builtin_nan("");
    }
    return;
  }
  if (status != kStatusOk) {
    if (threadIdx.x == 0) F_hat[p] = -__builtin_inf();
    for (int l = threadIdx.x; l < np; l += blockDim.x) {
      if (F_part) F_part[p * part_stride + l] = 0.0;
      if (amps)
        for (int i = 0; i < 4; ++i) amps[(p * part_stride + l) * 4 + i] = 0.0;
    }
    return;
  }
  for (int l = threadIdx.x >> 3; l < np; l += blockDim.x >> 3) {   // whole groups of eight
    const int64_t q = p * stride + l;
    double a[8], am[4];
    partition_sums(partials, off[q], cnt[q], k, a);
    const double F = solve_partition(a);
    if (amps) {
      double beta[4];
      solve_beta(a, beta);
      const double m = umax[0];
      amps_from_beta(P, beta, m > 0.0 ? sqrt(1.0 / m) : 1.0, am);
    }
    if (k != 0) continue;
    Fl[q] = F;
    if (F_part) F_part[p * part_stride + l] = F;
    if (amps)
      for (int i = 0; i < 4; ++i) amps[(p * part_stride + l) * 4 + i] = am[i];
  }
  __syncthreads();                             // Fl of this block's partitions
  if (threadIdx.x >= 64) return;
  double s = 0.0;
  for (int l = threadIdx.x; l < np; l += 64) s += Fl[p * stride + l];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (threadIdx.x == 0) {
    F_hat[p] = s / (double)np;
    if (bin_counter) atomicAdd(bin_counter, (unsigned long long)(P.j_hi - P.j_lo + 1));
  }
}

// ---------------------------------------------------------------------------
// template signal (for injections): sum_i a_i A^i with the full transfer
// ---------------------------------------------------------------------------
// f^{-7/6} = f^{-1/6} / f, the root from an FP32 estimate and one third-order step on
// f w^6 = 1 (its remainder, ~10 e^3, is below 1e-19), within two ulp
__device__ __forceinline__ double pow_m7_6(double f) {
  const double w = (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf((float)f) * (-1.0f / 6.0f));
  const double w2 = w * w;
  const double e = fma(-(w2 * w2), w2 * f, 1.0);
  return fma(w * e, fma(e, 7.0 / 72.0, 1.0 / 6.0), w) / f;
}

// One bin per thread and turn; 2048 blocks, so that the sine table and the particle's
// dropped phase are set up once per block.  Bound by FP64 issue (the template's phase in
// double-double): 7,101,001 bins 52 -> 30 us with the library's sines and power taken
// out (the stores alone need 24).
constexpr int kWaveBlocks = 2048;
__global__ __launch_bounds__(256) void k_waveform(Grid g, const PartConst* __restrict__ pc,
                                                  const double* __restrict__ amps,
                                                  double2* __restrict__ out) {
  __shared__ double2 s_tab[kSinTab];
  __shared__ double2 s_drop;
  const PartConst& P = pc[0];
  const bool ok = P.status == kStatusOk;
  if (ok) {
    // (formed here: a call needs no plan, whose creation fills the constant table)
    for (int i = threadIdx.x; i < kSinTab; i += blockDim.x) {
      double sv, cv;
      sincospi((double)i * (2.0 / (double)kSinTab), &sv, &cv);
      s_tab[i] = double2{sv, cv};
    }
    if (threadIdx.x == 0) {
      double sc, cc;
      sincospi(2.0 * dropped_phase(P), &sc, &cc);
      s_drop = double2{sc, cc};
    }
  }
  __syncthreads();
  const double sc = s_drop.x, cc = s_drop.y;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < g.nbins;
       j += (int64_t)gridDim.x * blockDim.x) {
    if (!ok || j < P.j_lo || j > P.j_hi) {
      out[j] = double2{0.0, 0.0};
      continue;
    }
    double f = bin_freq(g, j);
    double s0, c0;
    sincos_tab(0.5 * kLs * f, s_tab, s0, c0);
    double cph, sph, tpr, tpi, txr, txi;
    template_fp64(P, f, s0, c0, cph, sph, tpr, tpi, txr, txi, nullptr, g.chan.code[0], &g.orb, s_tab);
    // restore the constant phase the statistic drops
    double cps = cph * cc - sph * sc, sps = sph * cc + cph * sc;   // e^{i Phi_full}
    // full transfer: C(f) times the particle part T''
    double x0 = kPi * kLs * f;
    double zr = c0 * c0 - s0 * s0, zi = -2.0 * s0 * c0;
    double omr = 1.0 - (zr * zr - zi * zi), omi = -2.0 * zr * zi;
    double er = -x0 * s0, ei = -x0 * c0;
    double Cr = omr * er - omi * ei, Ci = omr * ei + omi * er;
    double Tpr = Cr * tpr - Ci * tpi, Tpi = Cr * tpi + Ci * tpr;
    double Txr = Cr * txr - Ci * txi, Txi = Cr * txi + Ci * txr;
    // h = f^{-7/6} e^{-i Phi} [(a1 - i a3) T+ + (-a2 + i a4) Tx]  (App. B basis)
    double a1 = amps[0], a2 = amps[1], a3 = amps[2], a4 = amps[3];
    double hr = (a1 * Tpr + a3 * Tpi) + (-a2 * Txr - a4 * Txi);
    double hi = (a1 * Tpi - a3 * Tpr) + (-a2 * Txi + a4 * Txr);
    const double amp = pow_m7_6(f);
    // multiply by e^{-i Phi} = cps - i sps
    out[j] = double2{amp * (hr * cps + hi * sps), amp * (hi * cps - hr * sps)};
  }
}

// ---------------------------------------------------------------------------
// extrinsic parameters from a_1..a_4 (App. B, Eq. extrinPara), one row per
// thread.  D_L = 2 / A and iota = arccos(-Ax / A) as printed.  For psi and
// phi_c the kernel uses the phases of the two circular parts of a,
//   (a1 + a4) + i (a2 - a3) = r1 e^{i (phi_c - 2 psi)},
//   (a1 - a4) - i (a2 + a3) = r2 e^{i (phi_c + 2 psi)},
// which give the same (psi, phi_c) as the printed arctangent ratios (whose
// arguments are 2 r1 r2 sin 2psi sin phi_c, 2 r1 r2 cos 2psi sin phi_c and
// 2 r1 r2 sin 2psi cos phi_c, read with the sign c = sgn(sin 2 psi)) and the
// same representative, phi_c in (0, pi] and psi in (-pi/2, pi/2], but stay
// accurate where those ratios approach 0/0.  At iota = 0 or pi one circular
// part vanishes (modulus below 64 ulp of the other) and only the other's
// phase is defined: psi = 0, phi_c = that phase.  All-zero a gives
// (inf, nan, nan, nan).  With the chirp mass (params != null) D_L is
// converted to metres with the App. A constant |A| D_L = sqrt(5/24)
// Mc^{5/6} / pi^{2/3} (geometric units), whose negative sign turns phi_c by pi.
// ---------------------------------------------------------------------------
__global__ void k_extrinsic(const double* __restrict__ amps, const double* __restrict__ params,
                            int64_t n, double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double a1 = amps[4 * i], a2 = amps[4 * i + 1], a3 = amps[4 * i + 2], a4 = amps[4 * i + 3];
  const double p1 = a1 + a4, p2 = a2 - a3, m1 = a1 - a4, m2 = -(a2 + a3);
  const double r1 = sqrt(p1 * p1 + p2 * p2), r2 = sqrt(m1 * m1 + m2 * m2);
  const double Ap = r1 + r2, Ax = r1 - r2;
  const double A = Ap + sqrt(fmax((Ap - Ax) * (Ap + Ax), 0.0));   // no cancellation at iota ~ 0
  double D, iota, psi, phic;
  if (!(A > 0.0)) {
    const double nan = __builtin_nan("");
    D = (A == 0.0) ? __builtin_inf() : nan;
    iota = psi = phic = nan;
  } else {
    D = 2.0 / A;
    iota = acos(fmin(fmax(-Ax / A, -1.0), 1.0));
    const double th1 = atan2(p2, p1);    // phi_c - 2 psi
    const double th2 = atan2(m2, m1);    // phi_c + 2 psi
    if (fmin(r1, r2) <= 64.0 * 2.220446049250313e-16 * fmax(r1, r2)) {
      psi = 0.0;
      phic = (r1 < r2) ? th2 : th1;
    } else {
      phic = 0.5 * (th1 + th2);          // (-pi, pi], defined modulo pi
      if (phic <= 0.0) phic += kPi;
      double d = th2 - phic;             // 2 psi, in (-2 pi, pi]
      if (d <= -kPi) d += 2.0 * kPi;
      psi = 0.5 * d;
    }
    if (params) {
      const double mc = params[6 * i + 1] * kMsunS;
      D *= kC * sqrt(5.0 / 24.0) * pow(mc, 5.0 / 6.0) / pow(kPi, 2.0 / 3.0);
      phic += (phic > 0.0) ? -kPi : kPi;
    }
  }
  out[4 * i] = D;
  out[4 * i + 1] = iota;
  out[4 * i + 2] = psi;
  out[4 * i + 3] = phic;
}

}  // namespace fstat

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
namespace fstat {

static inline unsigned nblk(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

void launch_prep(const Grid& g, const double* data, const double* psd, BinData<double> b,
                 hipStream_t s) {
  hipLaunchKernelGGL(k_prep, dim3(nblk(g.nbins, 256), g.chan.n), dim3(256), 0, s, g, data, psd, b.wr, b.wi,
                     b.u, b.s0, b.c0);
}

void launch_max(const double* u, int64_t n, double* out, hipStream_t s) {
  auto* bits = reinterpret_cast<unsigned long long*>(out);
  hipLaunchKernelGGL(k_zero64, dim3(1), dim3(64), 0, s, bits);
  hipLaunchKernelGGL(k_max, dim3(std::min<unsigned>(nblk(n, 2048), 512)), dim3(256), 0, s, u, n, bits);
}

void launch_scale(const Grid& g, const double* umax, BinData<double> b, BinData<float> b32,
                  hipStream_t s) {
  hipLaunchKernelGGL(k_scale, dim3(nblk(g.nbins, 256), g.chan.n), dim3(256), 0, s, g, umax, b.wr, b.wi, b.u,
                     b.s0, b.c0, b32.wr, b32.wi, b32.u, b32.s0, b32.c0);
}

void launch_setup(const Grid& g, const double* params, int64_t n,
                  const int32_t* np, int32_t np_uniform, int32_t stride, const Tiling& tl,
                  const uint8_t* skip, const WorkSpace& ws, hipStream_t s) {
  // one wavefront per block: a small batch spreads over the CUs
  hipLaunchKernelGGL(k_setup, dim3((unsigned)n), dim3(64), 0, s, g, params, n, np, np_uniform,
                     stride, tl, skip, ws.pc, ws.bounds, ws.cnt, ws.ptot(), ws.widen(n * stride));
}

void launch_worklist(int64_t n, int32_t stride, const Tiling& tl, int32_t nch, const WorkSpace& ws,
                     bool all_exact, hipStream_t s) {
  const int32_t ntiles = tl.ntiles * nch;
  const int64_t m = n * stride;
  const int32_t nb = (int32_t)((m + kScanBlock - 1) / kScanBlock);
  if (n <= kScanOnce) {
    hipLaunchKernelGGL(k_worklist, dim3((unsigned)n), dim3(256), 0, s, ws.cnt, ws.bounds,
                       ws.widen(m), stride, tl, nch, ws.ptot(), ws.off, ws.items, ws.total, ws.ndirect, ws.nrefine, all_exact ? 1 : 0,
                       ws.tcnt, ws.tcur, all_exact ? 0 : 2 * ntiles, ws.tile_ctr);
    return;
  }
  hipLaunchKernelGGL(k_scan_sums, dim3(nb), dim3(1024), 0, s, ws.cnt, m, ws.bsum);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, ws.bsum, nb, ws.total, ws.ndirect,
                     ws.nrefine);
  hipLaunchKernelGGL(k_scan_apply, dim3(nb), dim3(1024), 0, s, ws.cnt, m, ws.bsum, ws.off);
  hipLaunchKernelGGL(k_fill, dim3(nblk(m, 256)), dim3(256), 0, s, ws.cnt, ws.off, m, ws.bounds,
                     ws.widen(m), stride, tl, nch, ws.items);
  if (all_exact)
    hipLaunchKernelGGL(k_copy_count, dim3(1), dim3(64), 0, s, ws.total, ws.ndirect);
  else
    hipLaunchKernelGGL(k_tile_zero, dim3(nblk(2 * ntiles, 256)), dim3(256), 0, s, ws.tcnt, ws.tcur,
                       2 * ntiles, ws.tile_ctr);
}

Tiling make_tiling(const Grid& g, int32_t chunk, bool widen, bool mixed) {
  Tiling tl;
  tl.T = chunk;
  tl.rT = 1.0 / (double)chunk;
  tl.ntiles = (int32_t)((g.nbins + chunk - 1) / chunk);
  if (widen) {
    tl.mmax = std::max(1, std::min(kMaxWiden, (mixed ? kWidenMixed : kWidenFp64) / chunk));
    const double w = (double)chunk * g.df;          // [Hz] per tile
    tl.kt = (float)((mixed ? kWidenTimeMixed : kWidenTimeFp64) /
                    (w * (5.0 / 96.0) * pow(kPi, -8.0 / 3.0)));
    tl.kf = (float)(kWidenBand / w);
    tl.kd = mixed ? 0.f : (float)(kWidenSpan / kWidenTimeFp64);
  }
  return tl;
}

int interp_max_tile(bool mixed) { return mixed ? kMaxTileMixed : kMaxTileFp64; }

void launch_eval(bool mixed, bool interp, double refine_budget, const Grid& g,
                 int64_t n_particles, int32_t stride, const Tiling& tl, const WorkSpace& ws,
                 BinData<double> b, BinData<float> b32, const double* ek, int blocks,
                 hipStream_t s, hipEvent_t* ev_main, const UModel& um,
                 const Spectra<double>& s64, const Spectra<float>& s32) {
  const int32_t* sel = nullptr;
  const int32_t* nsel = nullptr;
  if (interp) {
    const int32_t ntiles = tl.ntiles * g.chan.n;   // all channels
    // The block loop needs tiles of whole blocks (the items inside a partition
    // then have no partial ones).
    SpecShape sp{};
    const int32_t L = mixed ? s32.L : s64.L;
    if (L > 0 && tl.T % L == 0)
      sp = mixed ? SpecShape{L, s32.Q, s32.nslots, s32.nblk, kSpecPsiMixed, 0.5 / s32.Q,
                             (double)(s32.nslots - 1) / s32.Q, s32.fmax}
                 : SpecShape{L, s64.Q, s64.nslots, s64.nblk, kSpecPsiFp64, 0.5 / s64.Q,
                             (double)(s64.nslots - 1) / s64.Q, s64.fmax};
    {
      const bool tab = g.orb.coef != nullptr;
      auto nodes = mixed ? (tab ? k_interp_nodes<true, true> : k_interp_nodes<true, false>)
                         : (tab ? k_interp_nodes<false, true> : k_interp_nodes<false, false>);
      hipLaunchKernelGGL(nodes, dim3(8 * blocks), dim3(256), 0, s, g, ws.pc, ws.bounds, stride,
                         ws.items, ws.total, tl, ek, ws.rec, ws.xflag, ws.xerr, ws.direct,
                         ws.ndirect, um, ws.partials, sp, 1.0 / (double)stride);
    }
    if (n_particles * (int64_t)(ntiles + stride * g.chan.n) <= kGroupOnce && 2 * ntiles <= kTileHist) {
      hipLaunchKernelGGL(k_tile_group, dim3(1), dim3(1024), 0, s, ws.items, ws.total, ws.xflag,
                         ntiles, ws.toff, ws.uoff,
                         ws.tile_items);
    } else {
      hipLaunchKernelGGL(k_tile_count, dim3(256), dim3(1024), 0, s, ws.items, ws.total, ws.xflag,
                         ntiles, ws.tcnt);
      hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(1024), 0, s, ws.tcnt, ntiles, ws.toff, ws.uoff);
      hipLaunchKernelGGL(k_tile_scatter, dim3(256), dim3(1024), 0, s, ws.items, ws.total, ws.xflag,
                         ntiles, ws.toff, ws.tcur,
                         ws.tile_items);
    }
    if (ev_main) (void)hipEventRecord(ev_main[0], s);
    if (sp.L > 0) {
      const int64_t ng = (int64_t)n_particles * stride * g.chan.n;
      const int eb = (int)std::min<int64_t>((2 * ng + 15) / 16, 8 * (int64_t)blocks);
      const int bb = (8 * blocks + 7) & ~7;      // a multiple of the XCD count
      if (mixed) {
        hipLaunchKernelGGL(k_eval_blocks<true>, dim3(bb), dim3(256), 0, s, s32, ws.tile_items,
                           ws.toff + ntiles, ws.rec, ws.partials);
        hipLaunchKernelGGL(k_eval_edges<true>, dim3(eb), dim3(256), 0, s, g, sp.L, sp.nblk, ng,
                           ws.cnt, ws.off, ws.xflag, b32.wr, b32.wi, ws.rec, ws.partials);
      } else {
        hipLaunchKernelGGL(k_eval_blocks<false>, dim3(bb), dim3(256), 0, s, s64, ws.tile_items,
                           ws.toff + ntiles, ws.rec, ws.partials);
        hipLaunchKernelGGL(k_eval_edges<false>, dim3(eb), dim3(256), 0, s, g, sp.L, sp.nblk, ng,
                           ws.cnt, ws.off, ws.xflag, b.wr, b.wi, ws.rec, ws.partials);
      }
    }
    // w (and e_j on the FP64 path) at the largest tile's stride
    const size_t lds = mixed ? (size_t)kMaxTileMixed * 2 * sizeof(float)
                             : (size_t)kMaxTileFp64 * (2 * sizeof(double) + sizeof(float));
    hipLaunchKernelGGL(mixed ? k_eval_interp<true> : k_eval_interp<false>, dim3(blocks), dim3(256),
                       lds, s, g, tl, ws.tile_items, ws.toff + ntiles, ws.uoff, ntiles,
                       ws.tile_ctr, b.wr, b.wi, b32.wr, b32.wi, ws.rec, ws.partials);
    if (ev_main) (void)hipEventRecord(ev_main[1], s);
    sel = ws.direct;
    nsel = ws.ndirect;
  }
  auto exact_pass = [&](const int32_t* list, const int32_t* count) {
    hipLaunchKernelGGL(mixed ? k_eval_exact<true> : k_eval_exact<false>, dim3(blocks), dim3(256),
                       0, s, g, ws.pc, ws.bounds, stride, ws.items, ws.total, tl, b.wr, b.wi,
                       b.u, b32.wr, b32.wi, b32.u, b.s0, b.c0, ek, ws.rec, ws.partials, list, count);
  };
  if (!interp && ev_main) (void)hipEventRecord(ev_main[0], s);
  exact_pass(sel, nsel);
  if (!interp && ev_main) (void)hipEventRecord(ev_main[1], s);
  if (interp && !mixed && refine_budget > 0.0) {
    // the mixed path's bar (1e-4 + 1e-6 cond) already covers the interpolation error
    const int64_t m = (int64_t)n_particles * stride;
    hipLaunchKernelGGL(k_mark, dim3(nblk(8 * m, 256)), dim3(256), 0, s, g,
                       s64.L > 0 ? spec_grid(g, s64.Q) : 0.0, ws.pc,
                       n_particles, ws.bounds, stride, ws.cnt, ws.off, ws.partials, ws.xflag,
                       ws.xerr, refine_budget, ws.refine, ws.nrefine);
    exact_pass(ws.refine, ws.nrefine);
  }
}

void launch_solve_mean(int64_t n, int32_t stride, const WorkSpace& ws, double* F_hat,
                       double* F_part, double* amps, int64_t part_stride, const double* umax,
                       unsigned long long* bin_counter, hipStream_t s) {
  // eight lanes for each of the particle's partitions, up to 128 at a time
  const unsigned bs = (unsigned)std::min((stride + 7) / 8, 16) * 64;
  hipLaunchKernelGGL(k_solve, dim3((unsigned)n), dim3(bs), 0, s, ws.pc, stride,
                     ws.cnt, ws.off, ws.partials, ws.Fl, F_hat, F_part, part_stride, amps, umax,
                     bin_counter);
}

void launch_sur_data(uint64_t seed, int64_t n, float* X, float* T, hipStream_t s) {
  hipLaunchKernelGGL(k_sur_data, dim3(nblk(n, 128)), dim3(128), 0, s, seed, n, X, T);
}

void launch_sur_knots(const Grid& g, int32_t stride, int64_t n, int64_t rows, const WorkSpace& ws,
                      float* X, hipStream_t s) {
  hipLaunchKernelGGL(k_sur_knots, dim3(nblk(rows, 256)), dim3(256), 0, s, g, ws.pc, ws.bounds,
                     stride, n, rows, X);
}

void launch_sur_check(const Grid& g, int32_t stride, int64_t n, const WorkSpace& ws,
                      const float* ynn, double* ek, double* mm, double thr,
                      unsigned long long* counters, hipStream_t s) {
  hipLaunchKernelGGL(k_sur_check, dim3(nblk(n * stride, 128)), dim3(128), 0, s, g, ws.pc,
                     ws.bounds, stride, n, ynn, ek, mm);
  hipLaunchKernelGGL(k_sur_decide, dim3(nblk(n, 128)), dim3(128), 0, s, ws.pc, n, stride, mm, thr,
                     counters);
}

int uprefix_block_sums(int64_t n) { return (int)((n + kScanBlock - 1) / kScanBlock); }

void launch_uprefix(const double* u, int64_t n, double* bsum, double* out, hipStream_t s) {
  const int32_t nb = uprefix_block_sums(n);
  hipLaunchKernelGGL(k_uscan_sums, dim3(nb), dim3(1024), 0, s, u, n, bsum);
  hipLaunchKernelGGL(k_uscan_top, dim3(1), dim3(1024), 0, s, bsum, nb);
  hipLaunchKernelGGL(k_uscan_apply, dim3(nb), dim3(1024), 0, s, u, n, bsum, out);
}

void launch_ufit(const double* u, int64_t nbins, int32_t ntiles, double* coef, double* resid,
                 hipStream_t s) {
  if (ntiles > 0)
    hipLaunchKernelGGL(k_ufit, dim3(ntiles), dim3(kUTile), 0, s, u, nbins, ntiles, coef, resid);
}

void launch_extrinsic(const double* amps, const double* params, int64_t n, double* out,
                      hipStream_t s) {
  hipLaunchKernelGGL(k_extrinsic, dim3(nblk(n, 256)), dim3(256), 0, s, amps, params, n, out);
}

void launch_waveform(const Grid& g, const PartConst* pc, const double* amps,
                     double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_waveform, dim3(std::min<unsigned>(nblk(g.nbins, 256), kWaveBlocks)), dim3(256),
                     0, s, g, pc, amps, reinterpret_cast<double2*>(out));
}

}  // namespace fstat

namespace fstat {
hipError_t occupancy_fp64(int* blocks_per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_eval_exact<false>, 256, 0);
}
hipError_t occupancy_mixed(int* blocks_per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_eval_exact<true>, 256, 0);
}
}  // namespace fstat
