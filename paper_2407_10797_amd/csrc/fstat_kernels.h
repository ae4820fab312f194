// fstat_kernels.h -- host-side launchers of the libfstat kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fstat_internal.h"

namespace fstat {

// frequency grid f_j = (k_lo + j) df, j < nbins; support window [0, T_obs]
// TDI channels: 0 X, 1 Y, 2 Z (first-generation Michelson at spacecraft 1, 2,
// 3), 3 A = (Z - X)/sqrt 2, 4 E = (X - 2Y + Z)/sqrt 6, 5 T = (X + Y + Z)/sqrt 3.
constexpr int kMaxChannels = 6;
struct Channels {
  int32_t n = 1;                                  // channels summed by the statistic
  int32_t code[kMaxChannels] = {0, 0, 0, 0, 0, 0};   // channel codes in data order
};

struct Grid {
  double df;
  double T_obs;
  int64_t k_lo;
  int64_t nbins;       // bins per channel
  Channels chan{};     // per-channel arrays are stacked channel-major
  OrbitTable orb{};    // spacecraft orbit (analytic unless a table is set)
};

// per-bin prepared data of one precision (structure of arrays)
template <typename T>
struct BinData {
  T* wr;   // Re w_j
  T* wi;   // Im w_j
  T* u;    // u_j
  T* s0;   // sin(pi f_j L)
  T* c0;   // cos(pi f_j L)
};

struct WorkSpace {
  PartConst* pc;      // [n]
  int32_t* bounds;    // [n][stride + 1]
  int32_t* cnt;       // [n][stride]
  int32_t* off;       // [n][stride]
  int32_t* total;     // [1]
  int32_t* bsum;      // [ceil(n stride / 4096)] block sums of the count scan
  int2* items;        // [capacity]
  double* partials;   // [capacity][8]
  double* Fl;         // [n][stride]
  int32_t* direct;    // [capacity] items the interpolating kernel hands to the exact kernel
  int32_t* ndirect;   // [1]
  int32_t* tcnt;      // [2 tiles] items per bin tile: those of the block spectra, then those
                      // of the per-bin loop
  int32_t* tcur;      // [2 tiles] scatter cursors
  int32_t* toff;      // [2 tiles + 1] first item of each in tile_items
  int32_t* uoff;      // [tiles + 1] first scheduling unit of each tile (per-bin loop)
  int32_t* tile_items;  // [capacity] item indices grouped by loop and bin tile
  int32_t* tile_ctr;  // [1] next unit to take (dynamic schedule)
  uint8_t* xflag;     // [capacity] kItemBins, kItemExact or kItemBlocks
  double* rec;        // [capacity][kInterpRec] per-item interpolation records
  float2* xerr;       // [capacity] interpolation error of each interpolated item:
                      // x template (norm-weighted), y M-term quadrature (absolute)
  int32_t* refine;    // [capacity] interpolated items of ill-conditioned partitions
  int32_t* nrefine;   // [1]
  // items per particle [n]: kept where Fl is written at the evaluation's end
  int32_t* ptot() const { return reinterpret_cast<int32_t*>(Fl); }
  // tiles per work item of each partition [n * stride], likewise (n <= n * stride)
  int32_t* widen(int64_t m) const { return reinterpret_cast<int32_t*>(Fl) + m; }
};

// How partitions are cut into work items: at the edges of tiles of T bins, or, where
// mmax > 1, of m consecutive tiles with m chosen per partition (item_width).
struct Tiling {
  int32_t T = 0, ntiles = 0;        // bins per tile, tiles of one channel
  double rT = 0.0;                  // 1 / T
  int32_t mmax = 1;                 // at most kMaxWiden
  float kt = 0.f, kf = 0.f;         // limits of m: kt Mc^{5/3} f^{11/3}, kf f
  float kd = 0.f;                   // shortest partition that is widened (in tiles, over the first limit)
};
constexpr int kMaxWiden = 7;        // an item's m in three bits beside its tile
Tiling make_tiling(const Grid& g, int32_t chunk, bool widen, bool mixed);

void launch_prep(const Grid& g, const double* data, const double* psd, BinData<double> b,
                 hipStream_t s);
void launch_max(const double* u, int64_t n, double* out, hipStream_t s);
void launch_scale(const Grid& g, const double* umax, BinData<double> b, BinData<float> b32,
                  hipStream_t s);
void launch_setup(const Grid& g, const double* params, int64_t n,
                  const int32_t* np, int32_t np_uniform, int32_t stride, const Tiling& tl,
                  const uint8_t* skip, const WorkSpace& ws, hipStream_t s);
// all_exact: the exact loop takes every item
void launch_worklist(int64_t n, int32_t stride, const Tiling& tl, int32_t nch, const WorkSpace& ws,
                     bool all_exact, hipStream_t s);
int interp_tables_init();
constexpr int kMaxTileFp64 = 2560;   // largest tile (bins) of the LDS-staged loops
constexpr int kMaxTileMixed = 4608;   // FP32 w: 36 KB + 2 KB per block, four blocks per CU
int interp_max_tile(bool mixed);   // largest tile (bins) the LDS-staged loop accepts
constexpr int kInterpRec = 57;     // doubles per interpolation record
// WorkSpace::xflag: which loop evaluates an item
enum : uint8_t { kItemBins = 0, kItemExact = 1, kItemBlocks = 2 };

// Block spectra of the plan's data (see spectra.hip): for every block of L
// consecutive bins of a channel, nslots phase slopes q / Q [cycles per bin]
// and kSpecNodes complex node weights per slope:
// S[channel][block][slope][kSpecNodes][re, im].
constexpr int kSpecNodes = 16;
template <typename T>
struct Spectra {
  T* S = nullptr;
  int32_t L = 0;         // bins per block (a power of two); 0: no spectra
  int32_t Q = 0;         // slopes per cycle
  int32_t nslots = 0;    // slopes kept: 0 .. T_obs df Q
  int32_t nblk = 0;      // whole blocks per channel
  double fmax = 0.0;     // items that reach this frequency take the per-bin loop
  // values per channel
  size_t values() const { return (size_t)nblk * (size_t)nslots * 2 * kSpecNodes; }
};
// Default tile of a plan with spectra, and how far a partition's items may be
// widened: as long as the signal's time in an item stays below kWidenTime and its
// bandwidth below kWidenBand of the frequency, up to kWiden bins.  Longer items
// spread a node evaluation over more bins until the degree-9 interpolants miss
// their end points and the exact loop takes the item, and until the spectra of the
// blocks that items of one place are at together no longer fit an L2 (7680 bins
// FP64: 3.9 MB; block loop 1.26 -> 1.67 ms).  Np = 64 on 7.1M bins FP64, one channel,
// three channels, orbit table, ms: one tile of 2560 each 3.17, 2.65, 1.28; 7 days 2.95,
// 2.40, 1.29; 9 days 2.88, 2.45, 1.25; 14 days 3.85, 5.20, 1.47; 7 days and 7680 bins
// 3.18, 2.51, 1.38.  Mixed, the same batch and the first stage's: one tile of 5120 1.69,
// 2.61; tiles of 2560 and 12 days 1.69, 2.63; 15 days 1.62, 2.46; 20 days 1.80, 2.57.
// FP64 partitions that the signal spends less than kWidenSpan in are not widened: over
// so short a time the transfers T+ and Tx are nearly proportional, the partition is
// ill-conditioned and the longer items' end points say less about it (4096 x 256:
// 21 partitions beyond the refinement budget without this rule, 6 at two days, 1 at four
// as with one tile per item).
constexpr int kSpecChunkFp64 = 2560;
constexpr int kSpecChunkMixed = 2560;
constexpr int kWidenFp64 = 5120;
constexpr int kWidenMixed = 7680;
constexpr double kWidenTimeFp64 = 9.0 * 86400.0;     // [s]
constexpr double kWidenTimeMixed = 15.0 * 86400.0;
constexpr double kWidenBand = 0.01;
constexpr double kWidenSpan = 4.0 * 86400.0;
constexpr double kSpecMaxSlope = 1.001;   // largest T_obs df [cycles per bin] with spectra
// Block size for a data set of nbins bins per channel, 0 for none.
int spectra_block(bool mixed, int64_t nbins);
int spectra_slots(const Grid& g, int32_t Q);
double spec_fmax(const Grid& g, int32_t Q, double budget);   // FP64: Spectra::fmax
int spectra_tables_init();              // the weights of all block sizes, once per device
// Spectra of one channel (w at wr, wi) into s64 and/or s32; with both they share L and
// t64 has the slopes of t32 at its even places.
void launch_spectra(const Grid& g, const double* wr, const double* wi,
                    const Spectra<double>& t64, const Spectra<float>& t32, double* s64, float* s32,
                    hipStream_t s);

// Smooth model of the template-independent weight u = 4 df f^{-7/3} |C|^2 / S
// (scaled): a degree-9 Chebyshev least-squares fit per u-tile of kUTile bins,
// with its largest relative residual on the tile's bins.  Items whose bins
// lie in tiles fitted to within kUFitTol get their M-terms (P, Q, R) by
// quadrature of the interpolated u |T|^2 products instead of a per-bin sum.
constexpr int kUTile = 256;
constexpr int kUCoef = 10;
constexpr double kUFitTol = 1e-13;
constexpr int kSsumMax = 8192;     // largest item length of the quadrature table
struct UModel {
  const double* coef = nullptr;        // [ntiles][kUCoef] Chebyshev coefficients
  const int32_t* bad_prefix = nullptr; // [ntiles + 1] count of unfit tiles before each
  const double* resid = nullptr;       // [ntiles] largest relative residual of each fit
  int32_t ntiles = 0;
  const double* ssum = nullptr;        // [5][kSsumMax + 1]: sum_m T_2i(s_m), s_m = 2m/(nb-1) - 1
  const double* upre = nullptr;        // [channels][nbins + 1] prefix sums of u
};
const double* cheb_sums_table();       // the current device's quadrature table (after init)
void launch_ufit(const double* u, int64_t nbins, int32_t ntiles, double* coef, double* resid,
                 hipStream_t s);
// prefix sums out[0..n] of u[0..n) (bsum: uprefix_block_sums(n) doubles of scratch)
int uprefix_block_sums(int64_t n);
void launch_uprefix(const double* u, int64_t n, double* bsum, double* out, hipStream_t s);
void launch_eval(bool mixed, bool interp, double refine_budget, const Grid& g,
                 int64_t n_particles, int32_t stride, const Tiling& tl,
                 const WorkSpace& ws, BinData<double> b, BinData<float> b32, const double* ek,
                 int blocks, hipStream_t s, hipEvent_t* ev_main = nullptr,
                 const UModel& um = UModel{}, const Spectra<double>& s64 = Spectra<double>{},
                 const Spectra<float>& s32 = Spectra<float>{});
void launch_sur_data(uint64_t seed, int64_t n, float* X, float* T, hipStream_t s);
void launch_sur_knots(const Grid& g, int32_t stride, int64_t n, int64_t rows, const WorkSpace& ws,
                      float* X, hipStream_t s);
void launch_sur_check(const Grid& g, int32_t stride, int64_t n, const WorkSpace& ws,
                      const float* ynn, double* ek, double* mm, double thr,
                      unsigned long long* counters, hipStream_t s);
// bins of the last evaluation by kind of interpolating-loop work, then the
// lane runs of those items by kind (out[kBinMix] accumulated)
constexpr int kBinMix = 14;
void launch_bin_mix(bool mixed, int32_t stride, const Tiling& tl, int32_t nch, const WorkSpace& ws,
                    unsigned long long* out, hipStream_t s);
void launch_solve_mean(int64_t n, int32_t stride, const WorkSpace& ws, double* F_hat,
                       double* F_part, double* amps, int64_t part_stride, const double* umax,
                       unsigned long long* bin_counter, hipStream_t s);
void launch_extrinsic(const double* amps, const double* params, int64_t n, double* out,
                      hipStream_t s);
void launch_waveform(const Grid& g, const PartConst* pc, const double* amps,
                     double* out, hipStream_t s);

}  // namespace fstat
