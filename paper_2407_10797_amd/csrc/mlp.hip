// mlp.hip -- learned surrogate for the eccentric phase correction Psi_e (App. A):
// a 3 -> 256 -> 256 -> 256 -> 256 -> 1 SiLU network, BF16 operands on MFMA with
// FP32 accumulation, FP32 master weights and Adam, trained on the GPU by the
// kernels below on samples produced by the plain template code.
//
// Parameter layout (flat FP32, 198,657 values):
//   W1[256][3] b1[256] | W2[256][256] b2[256] | W3 b3 | W4 b4 | w5[256] b5
// Inputs: (f, Mc, e0) mapped linearly to [-1, 1] over f in [10, 100] mHz,
// Mc in [10, 50] Msun, e0 in [0, 0.15].  Output: Psi_e / ((2355/1462) e0^2 Psi_N),
// the eccentric term in units of the factors the plain path computes anyway
// (e0^2 and the Newtonian phase), so that Psi_e = -(2355/1462) e0^2 Psi_N y.
#include <cmath>
#include <cstring>
#include <vector>

#include "../../include/fstat.h"
#include "fstat_api_internal.h"
#include "mlp.h"

namespace fstat {

typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// gfx950's 16x16x32 BF16 MFMA: lane l supplies A[l % 16][k] and B[k][l % 16]
// for its eight k of group l / 16 (the same k for A and B, so the order of k
// within a group does not matter), and receives D[4 (l / 16) + r][l % 16].
__device__ __forceinline__ v4f mfma32(v8s a, v8s b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                 __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

__device__ __forceinline__ uint16_t f2bf(float f) {   // round to nearest even
  return __builtin_bit_cast(uint16_t, (__bf16)f);       // v_cvt_pk_bf16_f32
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ float sigm(float z) { return 1.0f / (1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
// SiLU for the inference kernel: the reciprocal by the hardware's estimate and one
// Newton step, within 0.51 ulp, in 3 operations for the division's ~10
__device__ __forceinline__ float silu_nr(float z) {
  const float d = 1.0f + __expf(-z), r = __builtin_amdgcn_rcpf(d);
  const float q = fmaf(fmaf(-d, r, 1.0f), r, r);
  return z * (d < 3.0e38f ? q : 0.0f);                  // e^-z past FP32: 1 / inf
}
__device__ __forceinline__ float dsilu(float z) {
  float s = sigm(z);
  return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------
// Products of the training step, BF16 operands, FP32 accumulation.  Block = 4
// wavefronts = 64x64 outputs, each wave a 32x32 quadrant of 2x2 MFMA 16x16x32
// tiles.  K goes through LDS in panels: a panel's loads (16 bytes each) are all
// in flight at once and the MFMA steps run without a barrier between them, since
// a launch is bound by its rounds of load latency and not by bytes or products.
// M, N multiples of 64, K a multiple of 32 (checked by the host).
//
// A panel is kept in LDS as the MFMA fragments are read: 16 bytes = eight k of
// one row (m or n), the 64 rows of an octet of k side by side, row r of octet o
// at slot r ^ swz so that both the loads' stores and the fragment reads pass
// over all banks.
//   rows of memory are rows of the operand (H, dZ, W of the forward): swz = o % 8
//   rows of memory are k (dW's operands, W of dH): a thread transposes 8 x 8
//   values in registers; swz = (r / 8) % 8, which moves r within its group of 8
// ---------------------------------------------------------------------------
constexpr int kGemmK = 32;

__device__ __forceinline__ int slot_rows(int o, int r) { return o * 64 + (r ^ (o & 7)); }
__device__ __forceinline__ int slot_cols(int o, int r) { return o * 64 + (r ^ ((r >> 3) & 7)); }

// Rows r0 .. r0 + 63 of src[row][k], all kHid k, by 256 threads
struct RowPanel {
  uint4 v[8];
  __device__ __forceinline__ void load(const uint16_t* __restrict__ src, int r0, int t) {
    const int o = t & 31, r = t >> 5;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      v[i] = *reinterpret_cast<const uint4*>(src + (int64_t)(r0 + r + 8 * i) * kHid + 8 * o);
  }
  __device__ __forceinline__ void store(uint4* S, int t) const {
    const int o = t & 31, r = t >> 5;
#pragma unroll
    for (int i = 0; i < 8; ++i) S[slot_rows(o, r + 8 * i)] = v[i];
  }
};
// Rows r0 .. r0 + 63 of src[k][row]: thread t has octet t / 8 of k, from k0 on
struct ColPanel {
  uint4 v[8];
  __device__ __forceinline__ void load(const uint16_t* __restrict__ src, int r0, int k0, int t) {
    const int c = t & 7, o = t >> 3;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      v[i] = *reinterpret_cast<const uint4*>(src + (int64_t)(k0 + 8 * o + i) * kHid + r0 + 8 * c);
  }
  __device__ __forceinline__ void store(uint4* S, int t) const {
    const int c = t & 7, o = t >> 3;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      uint32_t w[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const uint32_t lo = q / 2 == 0 ? v[2 * h].x : q / 2 == 1 ? v[2 * h].y
                          : q / 2 == 2 ? v[2 * h].z : v[2 * h].w;
        const uint32_t hi = q / 2 == 0 ? v[2 * h + 1].x : q / 2 == 1 ? v[2 * h + 1].y
                          : q / 2 == 2 ? v[2 * h + 1].z : v[2 * h + 1].w;
        w[h] = q % 2 ? (lo >> 16) | (hi & 0xffff0000u) : (lo & 0xffffu) | (hi << 16);
      }
      S[slot_cols(o, 8 * c + q)] = uint4{w[0], w[1], w[2], w[3]};
    }
  }
};

// acc += the 32x32 quadrant (wr, wc) over octets of k [0, klen / 8) of two panels
template <bool ACOLS, bool BCOLS>
__device__ __forceinline__ void panel_mfma(const uint4* As, const uint4* Bs, int klen, int wr,
                                           int wc, int lane, v4f acc[2][2]) {
  const int rr = lane & 15;
  for (int kk = 0; kk < klen; kk += kGemmK) {
    const int o = (kk >> 3) + (lane >> 4);
    v8s b[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = 32 * wc + 16 * j + rr;
      b[j] = *reinterpret_cast<const v8s*>(&Bs[BCOLS ? slot_cols(o, r) : slot_rows(o, r)]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 32 * wr + 16 * i + rr;
      const v8s a = *reinterpret_cast<const v8s*>(&As[ACOLS ? slot_cols(o, r) : slot_rows(o, r)]);
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mfma32(a, b[j], acc[i][j]);
    }
  }
}

// First layer 3 -> 256 (VALU) for rows r0 .. r0 + 63 into the operand panel:
// z1 = W1 x + b1, h1 = bf16(SiLU(z1)); columns n0 .. n0 + 63 also to z1 and h1.
// All four column blocks of a row block form the same values: 11.0 us with the
// product, which a launch of its own (5.3 us) and the plain product (5.2) equal.
__device__ __forceinline__ void layer_in(const float* __restrict__ x, const float* __restrict__ W1,
                                         const float* __restrict__ b1, int r0, int n0,
                                         float* __restrict__ z1, uint16_t* __restrict__ h1,
                                         uint4* S) {
  const int o = threadIdx.x & 31, r = threadIdx.x >> 5;
  float w[8][3], bb[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    bb[e] = b1[8 * o + e];
#pragma unroll
    for (int q = 0; q < 3; ++q) w[e][q] = W1[(8 * o + e) * 3 + q];
  }
  const bool put = 8 * o >= n0 && 8 * o < n0 + 64;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int m = r0 + r + 8 * i;
    const float x0 = x[(int64_t)m * 3], x1 = x[(int64_t)m * 3 + 1], x2 = x[(int64_t)m * 3 + 2];
    float z[8];
    uint32_t p[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = bb[e] + w[e][0] * x0 + w[e][1] * x1 + w[e][2] * x2;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      p[e] = (uint32_t)f2bf(silu(z[2 * e])) | ((uint32_t)f2bf(silu(z[2 * e + 1])) << 16);
    const uint4 hv{p[0], p[1], p[2], p[3]};
    S[slot_rows(o, r + 8 * i)] = hv;
    if (put) {
      const int64_t at = (int64_t)m * kHid + 8 * o;
      *reinterpret_cast<uint4*>(h1 + at) = hv;
      *reinterpret_cast<float4*>(z1 + at) = float4{z[0], z[1], z[2], z[3]};
      *reinterpret_cast<float4*>(z1 + at + 4) = float4{z[4], z[5], z[6], z[7]};
    }
  }
}

enum { kEpiFwd = 0, kEpiBack = 1 };

struct GemmIo {
  const uint16_t* A;       // [m][k]
  const uint16_t* B;       // FWD [n][k], BACK [k][n]
  float* C;                // FWD Z, BACK with SUMS = 0 dz
  const float* vec;        // FWD bias[n], BACK zprev[m][n]
  uint16_t* H;             // FWD activations, BACK dz in BF16 (may be null)
  const float* x;          // IN and SUMS = 4: the inputs [m][3]
  float* part;             // SUMS: column sums
  const float *W1, *b1;    // IN
  float* z1;
  uint16_t* h1;
};

// C[m][n] = sum_k A(m,k) B(k,n) with K = kHid, one panel.
//   FWD  z = acc + bias[n] -> Z[m][n] (FP32), H[m][n] = bf16(SiLU(z)); with IN the
//        operand is the first layer's output, formed here from x
//   BACK d = acc SiLU'(zprev[m][n]) -> bf16, and with SUMS the column sums over
//        the block's 64 rows of d (SUMS = 1) or of d x_0, d x_1, d x_2, d (4);
//        SUMS = 0: d in FP32 as well
// Batch 4096 (256 blocks): forward 18.0 -> 5.4 us, dH with its activation and sums
// 27.6 -> 6.3 us (2-byte loads, 32-wide steps of K between barriers, and separate
// activation and sum kernels before).
template <int EPI, int SUMS, bool IN>
__global__ __launch_bounds__(256) void k_gemm_bf16(GemmIo io) {
  __shared__ uint4 As[64 * kHid / 8];
  __shared__ uint4 Bs[64 * kHid / 8];
  constexpr bool BCOLS = EPI == kEpiBack;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int wr = w >> 1, wc = w & 1;
  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  // what the epilogue reads, under way with the panels: lane holds
  // D[4 (lane/16) + r][lane % 16] of each 16x16 tile
  float ev[2][2][4];
  if constexpr (EPI == kEpiBack) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          ev[i][j][r] = io.vec[(int64_t)(m0 + 32 * wr + 16 * i + 4 * (lane >> 4) + r) * kHid + n0 +
                               32 * wc + 16 * j + (lane & 15)];
  } else {
#pragma unroll
    for (int j = 0; j < 2; ++j) ev[0][j][0] = io.vec[n0 + 32 * wc + 16 * j + (lane & 15)];
  }
  if constexpr (IN) {
    layer_in(io.x, io.W1, io.b1, m0, n0, io.z1, io.h1, As);
    RowPanel pb;
    pb.load(io.B, n0, t);
    pb.store(Bs, t);
  } else if constexpr (BCOLS) {
    RowPanel pa;
    ColPanel pb;
    pa.load(io.A, m0, t);
    pb.load(io.B, n0, 0, t);
    pa.store(As, t);
    pb.store(Bs, t);
  } else {
    RowPanel pa, pb;
    pa.load(io.A, m0, t);
    pb.load(io.B, n0, t);
    pa.store(As, t);
    pb.store(Bs, t);
  }
  __syncthreads();
  panel_mfma<false, BCOLS>(As, Bs, kHid, wr, wc, lane, acc);
  float (*D)[65] = reinterpret_cast<float (*)[65]>(As);          // SUMS: the 64x64 tile of d
  if constexpr (EPI == kEpiBack && SUMS > 0) __syncthreads();    // As is read no more
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ml = 32 * wr + 16 * i + 4 * (lane >> 4) + r, nl = 32 * wc + 16 * j + (lane & 15);
        const int64_t at = (int64_t)(m0 + ml) * kHid + n0 + nl;
        const float v = acc[i][j][r];
        if constexpr (EPI == kEpiFwd) {
          const float z = v + ev[0][j][0];
          io.C[at] = z;
          io.H[at] = f2bf(silu(z));
        } else {
          const float d = v * dsilu(ev[i][j][r]);
          if (io.H) io.H[at] = f2bf(d);
          if constexpr (SUMS > 0) D[ml][nl] = d;
          else io.C[at] = d;
        }
      }
  if constexpr (EPI == kEpiBack && SUMS > 0) {
    float* red = reinterpret_cast<float*>(Bs);                   // [4][SUMS][64]
    const int c = t & 63, g = t >> 6;
    float xr[16][SUMS > 1 ? SUMS - 1 : 1];
    if constexpr (SUMS > 1) {
#pragma unroll
      for (int k = 0; k < 16; ++k)
#pragma unroll
        for (int q = 0; q < SUMS - 1; ++q) xr[k][q] = io.x[(int64_t)(m0 + g + 4 * k) * 3 + q];
    }
    __syncthreads();
    float sum[SUMS];
#pragma unroll
    for (int q = 0; q < SUMS; ++q) sum[q] = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) {                               // the order of k_colred
      const float v = D[g + 4 * k][c];
#pragma unroll
      for (int q = 0; q < SUMS; ++q) sum[q] = q < SUMS - 1 ? fmaf(v, xr[k][q], sum[q]) : sum[q] + v;
    }
#pragma unroll
    for (int q = 0; q < SUMS; ++q) red[(g * SUMS + q) * 64 + c] = sum[q];
    __syncthreads();
    if (g == 0) {
#pragma unroll
      for (int q = 0; q < SUMS; ++q)
        io.part[((int64_t)blockIdx.y * SUMS + q) * kHid + n0 + c] =
            red[q * 64 + c] + red[(SUMS + q) * 64 + c] + red[(2 * SUMS + q) * 64 + c] +
            red[(3 * SUMS + q) * 64 + c];
    }
  }
}

// Split-K partial products of dW_2..dW_4 in one launch: block z has split
// z % ks (kper rows of the batch) of layer z / ks, C[z][m][n] = sum_k A[k][m] B[k][n].
// Panels of 128 k, half of the block's threads loading each operand and the next
// panel's loads under way during the products: 32 KB of LDS, so that the 768
// blocks of a batch of 4096 are resident together.  3 x 15.3 -> 9.7 us (panels of
// 256 k, 64 KB of LDS: 11.9).
struct DwOps {
  const uint16_t* A[3];
  const uint16_t* B[3];
};
__global__ __launch_bounds__(256) void k_gemm_dw(DwOps op, int ks, int kper,
                                                 float* __restrict__ C) {
  constexpr int kPanel = 128;
  __shared__ uint4 S[2][64 * kPanel / 8];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int wr = w >> 1, wc = w & 1;
  const int layer = blockIdx.z / ks;
  const int kbeg = (blockIdx.z % ks) * kper, kend = kbeg + kper;
  const int mine = t >> 7, tp = t & 127;              // operand, thread within it
  const uint16_t* src = mine ? op.B[layer] : op.A[layer];
  const int r0 = mine ? n0 : m0, k8 = 8 * (tp >> 3);
  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  ColPanel p;
  if (kbeg + k8 < kend) p.load(src, r0, kbeg, tp);
  for (int k0 = kbeg; k0 < kend; k0 += kPanel) {
    if (k0 + k8 < kend) p.store(S[mine], tp);
    __syncthreads();
    if (k0 + kPanel + k8 < kend) p.load(src, r0, k0 + kPanel, tp);
    panel_mfma<true, true>(S[0], S[1], min(kPanel, kend - k0), wr, wc, lane, acc);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        C[(int64_t)blockIdx.z * kHid * kHid +
          (int64_t)(m0 + 32 * wr + 16 * i + 4 * (lane >> 4) + r) * kHid + n0 + 32 * wc + 16 * j +
          (lane & 15)] = acc[i][j][r];
}

// output layer 256 -> 1 (FP32 from the FP32 pre-activations), squared error,
// dy = 2 (y - t) / B.  One wavefront per sample.
__global__ void k_layer_out(const float* __restrict__ z4, int B, const float* __restrict__ w5,
                            const float* __restrict__ b5, const float* __restrict__ tgt,
                            float* __restrict__ y, float* __restrict__ dy,
                            float* __restrict__ sqerr) {
  int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, lane = threadIdx.x & 63;
  if (wave >= B) return;
  float s = 0.f;
  for (int k = lane; k < kHid; k += 64) s += w5[k] * silu(z4[(int64_t)wave * kHid + k]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) {
    float yy = s + b5[0];
    y[wave] = yy;
    if (tgt) {
      float e = yy - tgt[wave];
      dy[wave] = 2.0f * e / (float)B;
      sqerr[wave] = e * e;
    }
  }
}

// fixed-order sum of B values by one block
template <typename V>
__device__ __forceinline__ V block_sum(const float* __restrict__ v, int B, V* red) {
  V s = 0;
#pragma unroll 16
  for (int i = threadIdx.x; i < B; i += 256) s += (V)v[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  return red[0];
}

// dz4 = dy w5 * SiLU'(z4) (bf16) for 64 columns and
// the rows of slice blockIdx.y, with the slice's column sums of dy SiLU(z4) (dW5)
// and of dz4 (db4) in the order of k_colred.  Two blocks past the slices sum dy
// (db5) and the squared errors (the batch's mean loss, where loss is given).
// Batch 4096: 4.2 us; the six launches that this was took 43 us, 15.6 of them a
// single block's serial sum over the slices (now in k_adam, beside its other sums).
__global__ __launch_bounds__(256) void k_out_back(const float* __restrict__ z4, int B, int slices,
                                                  const float* __restrict__ w5,
                                                  const float* __restrict__ dy,
                                                  const float* __restrict__ sq,
                                                  uint16_t* __restrict__ dzb,
                                                  float* __restrict__ part5,
                                                  float* __restrict__ part4,
                                                  float* __restrict__ db5,
                                                  double* __restrict__ loss) {
  __shared__ double sred[256];
  if ((int)blockIdx.y == slices) {
    if (blockIdx.x == 0) {
      const float v = block_sum<float>(dy, B, reinterpret_cast<float*>(sred));
      if (threadIdx.x == 0) db5[0] = v;
    } else if (blockIdx.x == 1 && loss) {
      const double v = block_sum<double>(sq, B, sred);
      if (threadIdx.x == 0) loss[0] = v / (double)B;
    }
    return;
  }
  float (*red)[2][64] = reinterpret_cast<float (*)[2][64]>(sred);
  const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int n = blockIdx.x * 64 + c;
  const int rows = (B + slices - 1) / slices;
  const int m0 = blockIdx.y * rows, m1 = min(B, m0 + rows);
  const float w = w5[n];
  float a5 = 0.f, a4 = 0.f;
#pragma unroll 16
  for (int m = m0 + g; m < m1; m += 4) {
    const int64_t at = (int64_t)m * kHid + n;
    const float z = z4[at], dm = dy[m];
    a5 = fmaf(silu(z), dm, a5);
    const float d = dm * w * dsilu(z);
    dzb[at] = f2bf(d);
    {
#pragma clang fp contract(off)
      a4 = a4 + d;                       // of the rounded d, as every column sum
    }
  }
  red[g][0][c] = a5;
  red[g][1][c] = a4;
  __syncthreads();
  if (g == 0) {
    part5[(int64_t)blockIdx.y * kHid + n] = red[0][0][c] + red[1][0][c] + red[2][0][c] + red[3][0][c];
    part4[(int64_t)blockIdx.y * kHid + n] = red[0][1][c] + red[1][1][c] + red[2][1][c] + red[3][1][c];
  }
}

// Column reductions over the batch, in two fixed-order passes (no atomics):
// part[s][q][n] = sum over the rows m of slice s of a[m][n] * wq(m), where
// wq(m) = wv[m * wstride + q] for q < NW, 1 otherwise; grad_of sums the slices.
// Block = 64 columns x 4 row groups; grid = (256 / 64, slices).
constexpr int kRedSlices = 64;

template <int Q, int NW>
__global__ __launch_bounds__(256) void k_colred(const float* __restrict__ a, int B,
                                                const float* __restrict__ wv, int wstride,
                                                float* __restrict__ part) {
  __shared__ float red[4][Q][64];
  const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int n = blockIdx.x * 64 + c;
  const int rows = (B + gridDim.y - 1) / gridDim.y;
  const int m0 = blockIdx.y * rows, m1 = min(B, m0 + rows);
  float acc[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) acc[q] = 0.f;
  for (int m = m0 + g; m < m1; m += 4) {
    const float v = a[(int64_t)m * kHid + n];
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q] += q < NW ? v * wv[(int64_t)m * wstride + q] : v;
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) red[g][q][c] = acc[q];
  __syncthreads();
  if (g == 0) {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      part[((int64_t)blockIdx.y * Q + q) * kHid + n] =
          red[0][q][c] + red[1][q][c] + red[2][q][c] + red[3][q][c];
  }
}

// Split-K partial products of dW_2..dW_4 and slice sums of the other gradients
// of one step: what the gradient of parameter i is summed from, in fixed order.
constexpr int kSplitK = 16;
struct GradParts {
  const float* splitk;     // [3][ks][256][256]
  const float* part;       // red: dW5 | db4 | db3 | db2 (one set of slices each) | dW1, db1 (four)
  int ks, slices;
  const float* db5;
};
__device__ __forceinline__ float grad_of(const GradParts& p, int64_t i) {
  const float* src;
  int64_t step;
  int n;
  if (i == mlp_off_b(4)) return p.db5[0];
  int l = 0;
  while (l < 4 && i >= mlp_off_w(l + 1)) ++l;
  if (l >= 1 && l <= 3 && i < mlp_off_b(l)) {             // W_l, l = 1..3 (W2..W4)
    src = p.splitk + (int64_t)(l - 1) * p.ks * kHid * kHid + (i - mlp_off_w(l));
    step = (int64_t)kHid * kHid;
    n = p.ks;
  } else {
    const int64_t set = (int64_t)kRedSlices * kHid;
    n = p.slices;
    if (l == 4) {                                         // w5
      src = p.part + (i - mlp_off_w(4));
      step = kHid;
    } else if (l >= 1) {                                  // b_l
      src = p.part + (4 - l) * set + (i - mlp_off_b(l));
      step = kHid;
    } else {                                              // W1[n][q], b1[n]
      const int64_t j = i - mlp_off_w(0);
      const bool bias = i >= mlp_off_b(0);
      const int64_t q = bias ? 3 : j % 3, c = bias ? i - mlp_off_b(0) : j / 3;
      src = p.part + 4 * set + q * kHid + c;
      step = 4 * kHid;
    }
  }
  float s = 0.f;
#pragma unroll 16
  for (int k = 0; k < n; ++k) s += src[(int64_t)k * step];
  return s;
}
__global__ void k_grad(GradParts p, int64_t n, float* __restrict__ g) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && i != mlp_off_b(4)) g[i] = grad_of(p, i);
}

// Inference-only forward of the whole network on R rows, keeping no
// activations (knot evaluation).  One wavefront per 32 rows (two MFMA tiles), four
// per block; the weights pass through LDS in 16 KB k-slabs of 32 shared by the four
// waves, and a fragment that a wave reads serves both of its tiles (with one tile
// the fragment reads, 64 KB per slab and CU, bounded the kernel: 1.05 M rows
// 1.38 -> 1.18 ms; three and four tiles at one wave per SIMD 1.55 and 2.06).  Then
// bound by the activations' VALU work: with the reciprocal of silu_nr in place of a
// division and the hardware's BF16 rounding 0.98 ms.
// Layer 1 runs on the VALU straight into the MFMA A-operand layout
// (lane l: row l % 16, k = 32 kb + 8 (l / 16) + j); layers 2-4 are 16x16x32
// BF16 MFMA tiles over all 256 outputs with the weights' BF16 copies read from
// the LDS slabs in the B-operand layout (col l % 16, same k); between layers
// the 16x256 tile goes through the wave's own LDS rows to turn the D layout
// (row 4 (l / 16) + r, col l % 16) back into the A layout.  The output unit
// is a lane reduction.  Same operand rounding as the training forward: BF16
// hidden activations, FP32 last pre-activation, FP32 output layer.
constexpr int kInferTiles = 2;
__global__ __launch_bounds__(256, 2) void k_mlp_infer(const float* __restrict__ x, int64_t R,
                                                   const float* __restrict__ P,
                                                   const uint16_t* __restrict__ wbf,
                                                   float* __restrict__ y) {
  constexpr int MT = kInferTiles;
  __shared__ __align__(16) uint16_t T[4][16][kHid + 8];
  __shared__ __align__(16) uint16_t Ws[2][kHid][kGemmK + 8];   // two k-slabs of W (rows n, 32 k)
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c16 = lane & 15, g4 = lane >> 4;
  const int64_t r0 = ((int64_t)blockIdx.x * 4 + w) * (16 * MT);
  constexpr int NK = kHid / kGemmK;
  v8s a[MT][NK];
  {
    const float* W1 = P + mlp_off_w(0);
    const float* b1 = P + mlp_off_b(0);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int64_t row = r0 + 16 * t + c16 < R ? r0 + 16 * t + c16 : R - 1;
      const float x0 = x[row * 3 + 0], x1 = x[row * 3 + 1], x2 = x[row * 3 + 2];
#pragma unroll
      for (int kb = 0; kb < NK; ++kb)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int k = kGemmK * kb + 8 * g4 + j;
          float z = b1[k] + W1[3 * k] * x0 + W1[3 * k + 1] * x1 + W1[3 * k + 2] * x2;
          a[t][kb][j] = (short)f2bf(silu_nr(z));
        }
    }
  }
  v4f acc[MT][16];
  // W_l[n][k] in k-slabs of 32 (16 KB), staged in LDS once for the block's four
  // waves and double-buffered: slab kb + 1 is fetched while slab kb is used
  const int tid = threadIdx.x;                      // row n of W that this thread stages
  for (int L = 0; L < 3; ++L) {
    const uint16_t* W = wbf + (size_t)L * kHid * kHid;
    const float* bias = P + mlp_off_b(L + 1);
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int nt = 0; nt < 16; ++nt) acc[t][nt] = v4f{0.f, 0.f, 0.f, 0.f};
    {
      const uint4* src = reinterpret_cast<const uint4*>(W + (size_t)tid * kHid);
#pragma unroll
      for (int q = 0; q < 4; ++q) *reinterpret_cast<uint4*>(&Ws[0][tid][8 * q]) = src[q];
    }
    __syncthreads();
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
      uint4 nxt[4];
      if (kb + 1 < NK) {
        const uint4* src =
            reinterpret_cast<const uint4*>(W + (size_t)tid * kHid + kGemmK * (kb + 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) nxt[q] = src[q];
      }
#pragma unroll
      for (int nt = 0; nt < 16; ++nt) {
        const v8s b = *reinterpret_cast<const v8s*>(&Ws[kb & 1][16 * nt + c16][8 * g4]);
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t][nt] = mfma32(a[t][kb], b, acc[t][nt]);
      }
      if (kb + 1 < NK) {
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<uint4*>(&Ws[(kb + 1) & 1][tid][8 * q]) = nxt[q];
      }
      __syncthreads();
    }
    if (L < 2) {
      // the wave's own rows of T, one tile after the other
#pragma unroll
      for (int t = 0; t < MT; ++t) {
#pragma unroll
        for (int nt = 0; nt < 16; ++nt) {
          const float bn = bias[16 * nt + c16];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            T[w][4 * g4 + r][16 * nt + c16] = f2bf(silu_nr(acc[t][nt][r] + bn));
        }
        __builtin_amdgcn_wave_barrier();      // LDS operations of a wave complete in order
#pragma unroll
        for (int kb = 0; kb < NK; ++kb)
          a[t][kb] = *reinterpret_cast<const v8s*>(&T[w][c16][kGemmK * kb + 8 * g4]);
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  const float* w5 = P + mlp_off_w(4);
  const float* b4 = P + mlp_off_b(3);
  const float b5 = P[mlp_off_b(4)];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nt = 0; nt < 16; ++nt) {
      const int n = 16 * nt + c16;
      const float wn = w5[n], bn = b4[n];
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] += wn * silu_nr(acc[t][nt][r] + bn);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) s[r] += __shfl_xor(s[r], o, 64);
    if (c16 == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = r0 + 16 * t + 4 * g4 + r;
        if (m < R) y[m] = s[r] + b5;
      }
    }
  }
}

// the BF16 copies of W2..W4
__device__ __forceinline__ void put_bf16(int64_t i, float v, uint16_t* __restrict__ wbf) {
  for (int l = 0; l < 3; ++l) {
    const int64_t o = i - mlp_off_w(l + 1);
    if (o >= 0 && o < (int64_t)kHid * kHid) wbf[(int64_t)l * kHid * kHid + o] = f2bf(v);
  }
}

// Adam on the flat parameter vector, each thread summing its parameter's
// gradient from its parts; refreshes the BF16 copies of W2..W4.  Bound by the 12.6 MB
// of split products: 7.4 us, where Adam, three split sums and the column sums of
// five groups by one block each took 5.1 + 3 x 5.3 + 122.
__global__ void k_adam(float* __restrict__ p, GradParts gp, float* __restrict__ m,
                       float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                       float c1, float c2, uint16_t* __restrict__ wbf) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float gi = grad_of(gp, i);
  float mi = b1 * m[i] + (1.f - b1) * gi;
  float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  put_bf16(i, pi, wbf);
}

__global__ void k_to_bf16(const float* __restrict__ p, uint16_t* __restrict__ wbf) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kNParams) put_bf16(i, p[i], wbf);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static inline unsigned nb(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

int Mlp::alloc(int batch) {
  if (batch <= cap_batch && params) return FSTAT_OK;
  release_acts();
  int rc;
  auto A = [&](void** p, size_t bytes) { return hip_check(hipMalloc(p, bytes ? bytes : 1), "mlp alloc"); };
  if (!params) {
    if ((rc = A((void**)&params, sizeof(float) * kNParams))) return rc;
    if ((rc = A((void**)&grad, sizeof(float) * kNParams))) return rc;
    if ((rc = A((void**)&m1, sizeof(float) * kNParams))) return rc;
    if ((rc = A((void**)&m2, sizeof(float) * kNParams))) return rc;
    if ((rc = A((void**)&wbf, sizeof(uint16_t) * 3 * kHid * kHid))) return rc;
    if ((rc = A((void**)&red, sizeof(float) * kRedSlices * 8 * kHid))) return rc;
    if ((rc = A((void**)&splitk, sizeof(float) * 3 * kSplitK * kHid * kHid))) return rc;
  }
  size_t BH = (size_t)batch * kHid;
  for (int l = 0; l < 4; ++l) {
    if ((rc = A((void**)&z[l], sizeof(float) * BH))) return rc;
    if ((rc = A((void**)&h[l], sizeof(uint16_t) * BH))) return rc;
  }
  // FP32 dz only where the column sums need a pass of their own
  if (!fused_sums(batch) && (rc = A((void**)&dz, sizeof(float) * BH))) return rc;
  if ((rc = A((void**)&dzb, sizeof(uint16_t) * 3 * BH))) return rc;
  if ((rc = A((void**)&y, sizeof(float) * batch))) return rc;
  if ((rc = A((void**)&dy, sizeof(float) * batch))) return rc;
  if ((rc = A((void**)&sq, sizeof(float) * batch))) return rc;
  cap_batch = batch;
  return FSTAT_OK;
}

void Mlp::release_acts() {
  for (int l = 0; l < 4; ++l) {
    if (z[l]) (void)hipFree(z[l]);
    if (h[l]) (void)hipFree(h[l]);
    z[l] = nullptr; h[l] = nullptr;
  }
  for (void* p : {(void*)dz, (void*)dzb, (void*)y, (void*)dy, (void*)sq})
    if (p) (void)hipFree(p);
  dz = nullptr; dzb = nullptr; y = nullptr; dy = nullptr; sq = nullptr;
  cap_batch = 0;
}

void Mlp::release() {
  release_acts();
  for (void* p : {(void*)params, (void*)grad, (void*)m1, (void*)m2, (void*)wbf, (void*)red,
                  (void*)splitk, (void*)yinf})
    if (p) (void)hipFree(p);
  params = grad = m1 = m2 = red = splitk = yinf = nullptr;
  cap_inf = 0;
  wbf = nullptr;
}

int Mlp::infer_alloc(int64_t rows) {
  if (yinf && rows <= cap_inf) return FSTAT_OK;
  if (yinf) (void)hipFree(yinf);
  yinf = nullptr;
  cap_inf = 0;
  int rc = hip_check(hipMalloc((void**)&yinf, sizeof(float) * (rows > 0 ? rows : 1)), "mlp alloc");
  if (!rc) cap_inf = rows;
  return rc;
}

void Mlp::infer(const float* x, int64_t rows, hipStream_t s) {
  if (rows <= 0) return;
  hipLaunchKernelGGL(k_mlp_infer, dim3(nb(rows, 64 * kInferTiles)), dim3(256), 0, s, x, rows, params, wbf, yinf);
}

void Mlp::refresh_bf16(hipStream_t s) {
  hipLaunchKernelGGL(k_to_bf16, dim3(nb(kNParams, 256)), dim3(256), 0, s, params, wbf);
}

// forward on B rows of x (B multiple of 64); tgt may be NULL
void Mlp::forward(const float* x, const float* tgt, int B, hipStream_t s) {
  const float* P = params;
  for (int l = 1; l < 4; ++l) {
    // Z_l = H_{l-1} W_l^T + b_l; H_0 from x
    GemmIo io{};
    io.A = h[l - 1];
    io.B = wbf + (size_t)(l - 1) * kHid * kHid;
    io.C = z[l];
    io.vec = P + mlp_off_b(l);
    io.H = h[l];
    const dim3 grid(kHid / 64, B / 64);
    if (l == 1) {
      io.x = x;
      io.W1 = P + mlp_off_w(0);
      io.b1 = P + mlp_off_b(0);
      io.z1 = z[0];
      io.h1 = h[0];
      hipLaunchKernelGGL((k_gemm_bf16<kEpiFwd, 0, true>), grid, dim3(256), 0, s, io);
    } else {
      hipLaunchKernelGGL((k_gemm_bf16<kEpiFwd, 0, false>), grid, dim3(256), 0, s, io);
    }
  }
  hipLaunchKernelGGL(k_layer_out, dim3(nb((int64_t)B * 64, 256)), dim3(256), 0, s, z[3], B,
                     P + mlp_off_w(4), P + mlp_off_b(4), tgt, y, dy, sq);
}

// Backward after forward(x, tgt): leaves the parts of every gradient (grad_parts).
// One slice of the column sums is 64 rows, the rows of a dH block, up to a batch
// of 4096: the dH kernels then form them themselves (6.0 us; with k_colred over an
// FP32 dz 5.7 more), above that a slice is longer than a block, and k_colred does.
bool Mlp::fused_sums(int B) { return B <= 64 * kRedSlices; }

void Mlp::backward(const float* x, int B, double* loss, hipStream_t s) {
  const int sl = B / 64 < kRedSlices ? B / 64 : kRedSlices;
  int ks = kSplitK;
  while (ks > 1 && (B % (kGemmK * ks))) ks >>= 1;
  const size_t set = (size_t)kRedSlices * kHid, BH = (size_t)B * kHid;
  const bool fused = fused_sums(B);
  parts_slices = sl;
  parts_ks = ks;
  // dz4; dW5[k] = sum_m dy[m] SiLU(z4[m][k]), db4; db5 = sum_m dy[m]
  hipLaunchKernelGGL(k_out_back, dim3(kHid / 64, sl + 1), dim3(256), 0, s, z[3], B, sl,
                     params + mlp_off_w(4), dy, sq, dzb + 2 * BH, red, red + set,
                     grad + mlp_off_b(4), loss);
  for (int l = 3; l >= 1; --l) {
    // dH_{l-1} = dZ_l W_l, dz_{l-1} = dH_{l-1} SiLU'(z_{l-1}); the column sums
    // give db_{l-1}, or dW1 and db1
    GemmIo io{};
    io.A = dzb + (l - 1) * BH;
    io.B = wbf + (size_t)(l - 1) * kHid * kHid;
    io.C = dz;
    io.vec = z[l - 1];
    io.H = l > 1 ? dzb + (l - 2) * BH : nullptr;
    io.x = x;
    io.part = red + (size_t)(5 - l) * set;
    const dim3 grid(kHid / 64, B / 64), rgrid(kHid / 64, sl);
    if (!fused)
      hipLaunchKernelGGL((k_gemm_bf16<kEpiBack, 0, false>), grid, dim3(256), 0, s, io);
    else if (l > 1)
      hipLaunchKernelGGL((k_gemm_bf16<kEpiBack, 1, false>), grid, dim3(256), 0, s, io);
    else
      hipLaunchKernelGGL((k_gemm_bf16<kEpiBack, 4, false>), grid, dim3(256), 0, s, io);
    if (!fused && l > 1)
      hipLaunchKernelGGL((k_colred<1, 0>), rgrid, dim3(256), 0, s, dz, B, (const float*)nullptr, 0,
                         io.part);
    if (!fused && l == 1)
      hipLaunchKernelGGL((k_colred<4, 3>), rgrid, dim3(256), 0, s, dz, B, x, 3, io.part);
  }
  // dW_l = dZ_l^T H_{l-1}, l = 1..3; K = B in ks splits (16 blocks a layer would
  // not fill the chip)
  hipLaunchKernelGGL(k_gemm_dw, dim3(kHid / 64, kHid / 64, 3 * ks), dim3(256), 0, s,
                     DwOps{{dzb, dzb + BH, dzb + 2 * BH}, {h[0], h[1], h[2]}}, ks, B / ks, splitk);
}

// the gradient itself (flat layout) from its parts
void Mlp::gradient(hipStream_t s) {
  hipLaunchKernelGGL(k_grad, dim3(nb(kNParams, 256)), dim3(256), 0, s,
                     GradParts{splitk, red, parts_ks, parts_slices, grad + mlp_off_b(4)},
                     (int64_t)kNParams, grad);
}

void Mlp::adam(int t, float lr, hipStream_t s) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  hipLaunchKernelGGL(k_adam, dim3(nb(kNParams, 256)), dim3(256), 0, s, params,
                     GradParts{splitk, red, parts_ks, parts_slices, grad + mlp_off_b(4)}, m1, m2,
                     (int64_t)kNParams, lr, b1, b2, eps, c1, c2, wbf);
}

}  // namespace fstat

using namespace fstat;

extern "C" int fstat_mlp_grad(const float* params, const float* x, const float* t, int32_t B,
                              double* loss, float* grad, float* y_out) {
  if (!params || !x || !t || B < 64 || (B % 64) || !loss || !grad)
    return set_error(FSTAT_EINVAL, "fstat_mlp_grad: bad arguments (B must be a multiple of 64)");
  Mlp net;
  int rc = net.alloc(B);
  float *dx = nullptr, *dt = nullptr;
  if (!rc) rc = hip_check(hipMalloc(&dx, sizeof(float) * 3 * B), "alloc x");
  if (!rc) rc = hip_check(hipMalloc(&dt, sizeof(float) * B), "alloc t");
  hipStream_t s = nullptr;
  if (!rc) rc = hip_check(hipMemcpy(net.params, params, sizeof(float) * kNParams, hipMemcpyHostToDevice), "copy");
  if (!rc) rc = hip_check(hipMemcpy(dx, x, sizeof(float) * 3 * B, hipMemcpyHostToDevice), "copy");
  if (!rc) rc = hip_check(hipMemcpy(dt, t, sizeof(float) * B, hipMemcpyHostToDevice), "copy");
  if (!rc) {
    net.refresh_bf16(s);
    net.forward(dx, dt, B, s);
    net.backward(dx, B, nullptr, s);
    net.gradient(s);
    rc = hip_check(hipGetLastError(), "mlp launch");
  }
  std::vector<float> sq(B);
  if (!rc) rc = hip_check(hipMemcpy(grad, net.grad, sizeof(float) * kNParams, hipMemcpyDeviceToHost), "copy grad");
  if (!rc) rc = hip_check(hipMemcpy(sq.data(), net.sq, sizeof(float) * B, hipMemcpyDeviceToHost), "copy loss");
  if (!rc && y_out) rc = hip_check(hipMemcpy(y_out, net.y, sizeof(float) * B, hipMemcpyDeviceToHost), "copy y");
  if (!rc) {
    double l = 0.0;
    for (int i = 0; i < B; ++i) l += sq[i];
    *loss = l / B;
  }
  if (dx) (void)hipFree(dx);
  if (dt) (void)hipFree(dt);
  net.release();
  return rc;
}

extern "C" int fstat_mlp_forward(const float* params, const float* x, int64_t R, float* y) {
  if (!params || !x || !y || R < 1 || R > ((int64_t)1 << 31))
    return set_error(FSTAT_EINVAL, "fstat_mlp_forward: bad arguments");
  Mlp net;
  int rc = hip_check(hipMalloc((void**)&net.params, sizeof(float) * kNParams), "alloc params");
  if (!rc) rc = hip_check(hipMalloc((void**)&net.wbf, sizeof(uint16_t) * 3 * kHid * kHid), "alloc wbf");
  if (!rc) rc = net.infer_alloc(R);
  float* dx = nullptr;
  if (!rc) rc = hip_check(hipMalloc(&dx, sizeof(float) * 3 * R), "alloc x");
  hipStream_t s = nullptr;
  if (!rc) rc = hip_check(hipMemcpy(net.params, params, sizeof(float) * kNParams, hipMemcpyHostToDevice), "copy");
  if (!rc) rc = hip_check(hipMemcpy(dx, x, sizeof(float) * 3 * R, hipMemcpyHostToDevice), "copy");
  if (!rc) {
    net.refresh_bf16(s);
    net.infer(dx, R, s);
    rc = hip_check(hipGetLastError(), "mlp launch");
  }
  if (!rc) rc = hip_check(hipMemcpy(y, net.yinf, sizeof(float) * R, hipMemcpyDeviceToHost), "copy y");
  if (dx) (void)hipFree(dx);
  net.release();
  return rc;
}
