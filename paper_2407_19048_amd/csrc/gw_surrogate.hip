// Learned waveform surrogate for gfx950: reduced-basis targets generated by
// the plain IMR-form model, basis construction (binary64 Gram matrix on the
// GPU, symmetric eigen-decomposition on the host), a 4-256-256-256-128 MLP
// with bfloat16 MFMA forward and backward kernels (binary32 accumulation,
// binary32 master weights, AdamW), reconstruction of plus/cross polarisations
// from the predicted node values, and a noise-weighted mismatch kernel.
//
// Node grid: NN = 1024 points log-spaced in geometric frequency Mf over
// [2e-3, 0.2]; targets are the amplitude ratio A/A_N and the phase residual
// P - P_N (Newtonian amplitude and phase removed analytically).
// Coefficients = A^T phi(theta) + zstd * z + zmean, where phi are the PN
// phase coefficient functions (exact inside the TaylorF2 region) and z is the
// MLP output.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "gw_fft.hpp"
#include "gw_physics.hpp"
#include "gw_internal.hpp"
#include "gw_linalg.hpp"
#include "../../include/gwgen.h"

using namespace gw;
using gw::linalg::chol_solve;
using gw::linalg::sym_eig;

namespace {

constexpr int NN = 1024;       // nodes
constexpr int NBAS = 64;       // basis vectors per target
constexpr int NOUT = 2 * NBAS; // MLP outputs
constexpr int NFEAT = 9;       // skip-path features
constexpr int HID = 256;
constexpr int NLAYER = 4;
constexpr double MF_LO = 2.0e-3, MF_HI = 0.2;

__host__ __device__ inline int layer_in(int l) { return l == 0 ? 16 : HID; }   // input padded to 16
__host__ __device__ inline int layer_out(int l) { return l == NLAYER - 1 ? NOUT : HID; }

// ------------------------------------------------------------------- bf16
__device__ __forceinline__ uint16_t f2bf(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}
// two at a time (v_cvt_pk_bf16_f32, the same rounding to nearest even): x in the low half
__device__ __forceinline__ uint32_t f2bf2(float x, float y) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
}
// a / d for finite a and 1 <= d <= 2^126: the reciprocal's quotient corrected by
// its exact remainder (correctly rounded but for rare ties; a fifth of the
// instructions of a division that scales its operands)
__device__ __forceinline__ float div_ge1(float a, float d) {
  const float r = __builtin_amdgcn_rcpf(d), q = a * r;
  return __builtin_fmaf(__builtin_fmaf(-q, d, a), r, q);
}
// A hidden layer's argument z as silu and its derivative take it: within
// [-87.25, largest binary32 number], NaN kept.  There 1 + exp(-z) is at most
// 2^126, so that its reciprocal is normal, and a / d of div_ge1 is finite, so
// that its remainder is a number.  What the bounds cut off: silu(z) of z below
// -87.25 is -1.1e-36 instead of something between that and zero, and silu of
// an infinity becomes one again when it is rounded to bfloat16.  (A division's
// fix-up instruction behind each quotient kept two more values of it alive, and
// 59 registers spilled instead of 35: 48.9 us for the gradients of 8192 rows
// instead of 41.8.)
__device__ __forceinline__ float silu_range(float z) {
  return __builtin_elementwise_minimum(__builtin_elementwise_maximum(z, -87.25f), 0x1.fffffep127f);
}
__device__ __forceinline__ float one_plus_exp(float z) { return 1.f + __expf(-z); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// -------------------------------------------------------- targets at nodes
struct TargetArgs {
  DevCfg cf;
  const double* params;  // [12][B]
  int64_t B;
  float* ratio;          // [B][NN]
  float* dpsi;           // [B][NN]
  double* feat;          // [B][NFEAT]
};

// Plain IMR-form model at an arbitrary frequency: intrinsic phase [rad] and
// amplitude ratio to the Newtonian amplitude.
__device__ void model_at(const WfModel& w, double Ms, double f, double* P, double* ratio) {
  const double two_pi = 2.0 * kPi;
  if (f < w.ft || w.f_rd == 0.0) {
    const double v = cbrt(kPi * Ms * f), lnv = log(v);
    const double iv = 1.0 / v, iv5 = iv * iv * iv * iv * iv;
    const double p = w.a[0] + v * v * (w.a[2] + v * (w.a[3] + v * (w.a[4] + v * ((w.a[5] + w.b5 * lnv) +
                     v * ((w.a[6] + w.b6 * lnv) + v * w.a[7])))));
    *P = two_pi * p * iv5;
    *ratio = 1.0;
    return;
  }
  *P = two_pi * (w.mr_b0 + w.mr_b1 * f) + atan((f - w.f_rd) * w.inv_fdamp);
  // A_N(f) = A_t (f / f_t)^(-7/6)
  const double AN = w.At * pow(f / w.ft, -7.0 / 6.0);
  double A;
  if (f < w.f_rd) A = w.At * pow(f / w.ft, -2.0 / 3.0);
  else {
    const double d = f - w.f_rd;
    A = w.Ard * w.fdamp2 / (d * d + w.fdamp2);
  }
  *ratio = A / AN;
}

__global__ __launch_bounds__(256) void k_targets(TargetArgs a) {
  __shared__ WfModel w;
  __shared__ double Ms_s, eta_s;
  const int64_t b = blockIdx.x;
  if (threadIdx.x < kSetupLanes) wf_setup_column(a.params, a.B, b, a.cf, threadIdx.x, nullptr, &w);
  if (threadIdx.x == 0) {
    const double q = a.params[1 * a.B + b], mc = a.params[0 * a.B + b];
    const double eta = q / ((1.0 + q) * (1.0 + q));
    eta_s = eta;
    Ms_s = mc * pow(eta, -0.6) * kMsunSec;
    // features: PN coefficients times 3/(128 eta) (w.a are in revolutions)
    const double two_pi = 2.0 * kPi;
    double* ft = a.feat + b * NFEAT;
    ft[0] = two_pi * w.a[2];
    ft[1] = two_pi * w.a[3];
    ft[2] = two_pi * w.a[4];
    ft[3] = two_pi * w.a[5];
    ft[4] = two_pi * w.a[6];
    ft[5] = two_pi * w.a[7];
    ft[6] = two_pi * w.b5;
    ft[7] = two_pi * w.b6;
    ft[8] = 1.0;
  }
  __syncthreads();
  const double dlog = log(MF_HI / MF_LO) / double(NN - 1);
  for (int j = threadIdx.x; j < NN; j += 256) {
    const double Mf = MF_LO * exp(dlog * j);
    const double f = Mf / Ms_s;
    double P, ratio;
    model_at(w, Ms_s, f, &P, &ratio);
    const double v = cbrt(kPi * Mf);
    const double PN = 3.0 / (128.0 * eta_s * v * v * v * v * v);
    a.ratio[b * NN + j] = float(ratio);
    a.dpsi[b * NN + j] = float(P - PN);
  }
}

// ------------------------------------------------ column means and Gram
__global__ __launch_bounds__(256) void k_colmean(const float* X, int64_t n, double* mean) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= NN) return;
  double s = 0.0;
  for (int64_t i = 0; i < n; ++i) s += X[i * NN + j];
  mean[j] = s / double(n);
}

// G = (X - mu)^T (X - mu), binary64; 32x32 output tile per block, 256
// threads, each accumulating 4 entries; rows staged through LDS.
__global__ __launch_bounds__(256) void k_gram(const float* X, int64_t n, const double* mean, double* G) {
  __shared__ double sa[32][33], sb[32][33];
  const int bi = blockIdx.y * 32, bj = blockIdx.x * 32;
  const int t = threadIdx.x;
  const int ti = t / 8, tj = (t % 8) * 4;  // 32 rows x 8 groups of 4 columns
  double acc[4] = {0, 0, 0, 0};
  for (int64_t r0 = 0; r0 < n; r0 += 32) {
    for (int e = t; e < 32 * 32; e += 256) {
      const int rr = e / 32, cc = e % 32;
      const int64_t row = r0 + rr;
      const bool ok = row < n;
      sa[rr][cc] = ok ? double(X[row * NN + bi + cc]) - mean[bi + cc] : 0.0;
      sb[rr][cc] = ok ? double(X[row * NN + bj + cc]) - mean[bj + cc] : 0.0;
    }
    __syncthreads();
#pragma unroll 4
    for (int rr = 0; rr < 32; ++rr) {
      const double av = sa[rr][ti];
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] += av * sb[rr][tj + q];
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) G[int64_t(bi + ti) * NN + bj + tj + q] = acc[q];
}

// C[n][NBAS] = (X - mu) V^T, V [NBAS][NN] binary32.  64 rows x 64
// coefficients per 256-thread block (4 x 4 outputs per thread), the 1024-long
// reduction in chunks of 32 staged through LDS.
__global__ __launch_bounds__(256) void k_project_basis(const float* X, int64_t n, const double* mean,
                                                       const float* V, float* C, int ldc, int coff) {
  __shared__ float xs[32][64 + 4];  // [j][row]
  __shared__ float vs[32][64 + 4];  // [j][coef]
  const int64_t r0 = int64_t(blockIdx.x) * 64;
  const int t = threadIdx.x;
  const int tr = (t / 16) * 4, tc = (t % 16) * 4;
  float acc[4][4] = {};
  for (int j0 = 0; j0 < NN; j0 += 32) {
    for (int e = t; e < 64 * 32; e += 256) {
      const int rr = e / 32, jj = e % 32;
      const int64_t row = r0 + rr;
      xs[jj][rr] = row < n ? float(double(X[row * NN + j0 + jj]) - mean[j0 + jj]) : 0.f;
      vs[jj][rr] = V[rr * NN + j0 + jj];
    }
    __syncthreads();
#pragma unroll 8
    for (int jj = 0; jj < 32; ++jj) {
      float xa[4], va[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { xa[q] = xs[jj][tr + q]; va[q] = vs[jj][tc + q]; }
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = fmaf(xa[a], va[c], acc[a][c]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int64_t row = r0 + tr + a;
    if (row < n)
#pragma unroll
      for (int c = 0; c < 4; ++c) C[row * ldc + coff + tc + c] = acc[a][c];
  }
}

// Normal equations of the skip path: P = phi^T phi [NFEAT][NFEAT] and
// Q = phi^T C [NFEAT][NOUT], binary64; one block per output column (+1 for P).
__global__ __launch_bounds__(256) void k_normal_eq(const double* feat, const float* C, int64_t n, double* P, double* Q) {
  __shared__ double red[256];
  const int col = blockIdx.x;  // 0..NOUT-1: Q columns; NOUT..NOUT+NFEAT-1: P columns
  const int t = threadIdx.x;
  for (int fi = 0; fi < NFEAT; ++fi) {
    double s = 0.0;
    for (int64_t i = t; i < n; i += 256) {
      const double y = col < NOUT ? double(C[i * NOUT + col]) : feat[i * NFEAT + (col - NOUT)];
      s += feat[i * NFEAT + fi] * y;
    }
    red[t] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (t < w) red[t] += red[t + w];
      __syncthreads();
    }
    if (t == 0) {
      if (col < NOUT) Q[fi * NOUT + col] = red[0];
      else P[fi * NFEAT + (col - NOUT)] = red[0];
    }
    __syncthreads();
  }
}

// residual targets: Z = (C - phi A - zmean) / zstd;  mode 0 computes the
// residual into Z only (statistics pass), mode 1 standardises in place.
__global__ __launch_bounds__(256) void k_residual(const double* feat, const float* C, const float* A, int64_t n,
                                                  const float* zmean, const float* zstd, float* Z, int mode) {
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e >= n * NOUT) return;
  const int64_t i = e / NOUT;
  const int o = int(e % NOUT);
  if (mode == 0) {
    double s = 0.0;
    for (int fi = 0; fi < NFEAT; ++fi) s += feat[i * NFEAT + fi] * double(A[fi * NOUT + o]);
    Z[e] = float(double(C[e]) - s);
  } else {
    Z[e] = (Z[e] - zmean[o]) / zstd[o];
  }
}

__global__ __launch_bounds__(256) void k_colstats(const float* Z, int64_t n, int ncol, float* mean, float* stdv) {
  __shared__ double s1[256], s2[256];
  const int col = blockIdx.x, t = threadIdx.x;
  double a = 0, q = 0;
  for (int64_t i = t; i < n; i += 256) {
    const double v = Z[i * ncol + col];
    a += v;
    q += v * v;
  }
  s1[t] = a;
  s2[t] = q;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) { s1[t] += s1[t + w]; s2[t] += s2[t + w]; }
    __syncthreads();
  }
  if (t == 0) {
    const double m = s1[0] / double(n);
    const double var = fmax(s2[0] / double(n) - m * m, 0.0);
    mean[col] = float(m);
    stdv[col] = float(fmax(sqrt(var), 1e-6));
  }
}

// ------------------------------------------------------------- network
// 4-256-256-256-128 MLP on bf16 MFMA (16x16x16, binary32 accumulation, K in
// increasing steps of 16), 32 rows per 1024-thread workgroup through every
// layer: activations in LDS as bf16, each wave owning 16 columns (of the
// output layer, for one half of the rows).  At the training batch of 8192 that is one workgroup per CU;
// what bounds it is the 800 KB of weights each workgroup reads from L2 (forward
// and backward order), so they are stored as the MFMA operands' own fragments
// and read 1 KB per wave and load.
//
// Fragments (4 bf16 per lane, lane = c + 16 g): the operand's element
// (index along its rows or columns c, k = 4 g + r).  Two steps of 16 along k
// lie side by side, so that a lane reads 16 bytes.
typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kMlpRows = 32;
constexpr int kMlpThreads = 1024;
constexpr int kActStride = HID + 4;  // bf16 per LDS row: 8-byte reads of 16 rows hit 32 distinct banks
constexpr int kBiasCols = 3 * HID + NOUT;

__host__ __device__ constexpr int bias_col(int l) { return l * HID; }  // first column of layer l's bias gradient

// Position of W[k][n] (k < nin, n < nout) in the fragments of the product
// x W (contraction over k, 16 columns n a tile)
__host__ __device__ inline int frag_fwd(int nin, int k, int n) {
  const int lane = (n & 15) + 16 * ((k & 15) >> 2), ks = k >> 4;
  if (nin == 16) return ((n >> 4) * 64 + lane) * 4 + (k & 3);
  return (((n >> 4) * (nin / 32) + (ks >> 1)) * 64 + lane) * 8 + (ks & 1) * 4 + (k & 3);
}
// and of the product dz W^T (contraction over n, 16 rows k a tile)
__host__ __device__ inline int frag_bwd(int nout, int k, int n) {
  const int lane = (k & 15) + 16 * ((n & 15) >> 2), ks = n >> 4;
  return (((k >> 4) * (nout / 32) + (ks >> 1)) * 64 + lane) * 8 + (ks & 1) * 4 + (n & 3);
}

struct MlpArgs {
  // inputs: theta [B][4], or columns b0 .. of params [12][pB] (theta NULL)
  const float* theta;
  const double* params;
  int64_t pB, b0, B;
  float lo[4], hi[4];
  const uint16_t* wf[NLAYER];   // fragments of x W
  const uint16_t* wb[NLAYER];   // fragments of dz W^T (training; layers 1..)
  const float* bias[NLAYER];
  // inference
  uint16_t* h_last;             // [B][HID] last hidden layer, or NULL
  float* z_out;                 // [B][NOUT]
  // training: targets, and per 32 rows the fragments (two steps of 16 rows) of
  // every layer's input and output gradient, the bias gradients' column sums
  // and the squared error
  const float* y;               // [B][NOUT]
  uint4* hfrag[NLAYER];         // [blocks][nin / 16][64]
  uint4* dfrag[NLAYER];         // [blocks][nout / 16][64]
  float* bias_part;             // [blocks][kBiasCols]
  float* loss_part;             // [blocks]
};

// A wave's fragments of one layer's weights (K rows, one tile of 16 columns).
// They do not depend on the activations, so each layer's are requested before
// the product ahead of it; the workgroup's barriers wait for LDS only.
template <int K> struct MlpFrags {
  static constexpr int KS = K / 16, STEP = K == 16 ? 1 : 2;  // steps of 16, steps per load
  struct alignas(8 * STEP) Load { v4s s[STEP]; };
  Load q[KS / STEP];
  __device__ __forceinline__ void load(const uint16_t* w, int tile, int lane) {
    const Load* wp = reinterpret_cast<const Load*>(w) + tile * (KS / STEP) * 64 + lane;
#pragma unroll
    for (int kp = 0; kp < KS / STEP; ++kp) q[kp] = wp[kp * 64];
  }
};

// acc[i] = rows 16 (i0 + i) .. of the LDS matrix `in` times w, for NI halves i
template <int NI, int K>
__device__ __forceinline__ void mlp_product(const uint16_t (*in)[kActStride], const MlpFrags<K>& w, int i0, int lane,
                                            v4f* acc) {
#pragma unroll
  for (int i = 0; i < NI; ++i) acc[i] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < K / 16; ++ks) {
    constexpr int STEP = MlpFrags<K>::STEP;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const v4s af = *reinterpret_cast<const v4s*>(&in[16 * (i0 + i) + (lane & 15)][16 * ks + 4 * (lane >> 4)]);
      acc[i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af, w.q[ks / STEP].s[ks % STEP], acc[i], 0, 0, 0);
    }
  }
}

// A lane's rounded values of one tile (four rows of each of the two row
// halves): as a fragment pair and, in `out`, at their rows' column.
__device__ __forceinline__ uint4 frag_pair(const float (*x)[4]) {
  return uint4{f2bf2(x[0][0], x[0][1]), f2bf2(x[0][2], x[0][3]), f2bf2(x[1][0], x[1][1]), f2bf2(x[1][2], x[1][3])};
}
__device__ __forceinline__ void frag_to_rows(uint4 h, uint16_t (*out)[kActStride], int tile, int lane) {
  const uint32_t w[4] = {h.x, h.y, h.z, h.w};
  const int row = 4 * (lane >> 4), col = 16 * tile + (lane & 15);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[16 * (i >> 1) + row + 2 * (i & 1)][col] = uint16_t(w[i]);
    out[16 * (i >> 1) + row + 2 * (i & 1) + 1][col] = uint16_t(w[i] >> 16);
  }
}

// Hidden layer L: z = x W + b kept by the wave, silu(z) rounded to LDS (and to
// the next layer's input fragments).
template <int L, bool TRAIN, int K>
__device__ __forceinline__ void mlp_hidden(const MlpArgs& a, const uint16_t (*in)[kActStride], uint16_t (*out)[kActStride],
                                           const MlpFrags<K>& w, int lane, int tile, v4f* z) {
  const float b = a.bias[L][16 * tile + (lane & 15)];
  mlp_product<2>(in, w, 0, lane, z);
  float x[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      z[i][r] = silu_range(z[i][r] + b);
      x[i][r] = div_ge1(z[i][r], one_plus_exp(z[i][r]));
    }
  const uint4 h = frag_pair(x);
  frag_to_rows(h, out, tile, lane);
  if constexpr (TRAIN) a.hfrag[L + 1][(int64_t(blockIdx.x) * (HID / 16) + tile) * 64 + lane] = h;
}

// dz of layer L - 1 from dz of layer L (in LDS): dH = dz W^T, times silu'(z);
// its fragments, LDS rows (if another layer follows) and bias gradient sums.
template <int L, int K>
__device__ __forceinline__ void mlp_backward_layer(const MlpArgs& a, const uint16_t (*in)[kActStride],
                                                   uint16_t (*out)[kActStride], const MlpFrags<K>& w, int lane, int tile,
                                                   const v4f* z) {
  v4f dh[2];
  mlp_product<2>(in, w, 0, lane, dh);
  float g[2][4], sum = 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float zz = z[i][r];
      const float s = div_ge1(1.f, one_plus_exp(zz));
      g[i][r] = dh[i][r] * s * (1.f + zz * (1.f - s));
      sum += g[i][r];
    }
  const uint4 h = frag_pair(g);
  if constexpr (L > 1) frag_to_rows(h, out, tile, lane);
  a.dfrag[L - 1][(int64_t(blockIdx.x) * (HID / 16) + tile) * 64 + lane] = h;
  sum += __shfl_xor(sum, 16);
  sum += __shfl_xor(sum, 32);
  if (lane < 16) a.bias_part[int64_t(blockIdx.x) * kBiasCols + bias_col(L - 1) + 16 * tile + lane] = sum;
}

template <bool TRAIN>
__global__ __launch_bounds__(kMlpThreads) void k_mlp(MlpArgs a) {
  __shared__ uint16_t act[2][kMlpRows][kActStride];
  __shared__ float red[kMlpThreads / 64], bsum[NOUT];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t r0 = int64_t(blockIdx.x) * kMlpRows;
  MlpFrags<16> w0;
  MlpFrags<HID> w1, w2, w3, v2, v1;
  MlpFrags<NOUT> v3;
  w0.load(a.wf[0], wv, lane);
  w1.load(a.wf[1], wv, lane);
  if (t < kMlpRows * 16) {
    // x = 2 (theta - lo)/(hi - lo) - 1 for (M_c, q, chi1, chi2), zero pad
    const int r = t / 16, c = t % 16;
    const int64_t row = r0 + r;
    uint16_t h = 0;
    if (c < 4 && row < a.B) {
      const float v = a.theta ? a.theta[row * 4 + c] : float(a.params[c * a.pB + a.b0 + row]);
      h = f2bf(2.f * (v - a.lo[c]) / (a.hi[c] - a.lo[c]) - 1.f);
    }
    act[0][r][c] = h;
  }
  lds_barrier();
  if constexpr (TRAIN) {
    if (wv == 0) {
      uint32_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * (i >> 1) + 4 * (lane >> 4) + 2 * (i & 1);
        h[i] = uint32_t(act[0][row][lane & 15]) | uint32_t(act[0][row + 1][lane & 15]) << 16;
      }
      a.hfrag[0][int64_t(blockIdx.x) * 64 + lane] = uint4{h[0], h[1], h[2], h[3]};
    }
  }
  v4f z0[2], z1[2], z2[2], zo;
  mlp_hidden<0, TRAIN>(a, act[0], act[1], w0, lane, wv, z0);
  w2.load(a.wf[2], wv, lane);
  lds_barrier();
  mlp_hidden<1, TRAIN>(a, act[1], act[0], w1, lane, wv, z1);
  // output layer: tile wv % 8 for the rows of half wv / 8
  const int tile = wv & 7, half = wv >> 3, col = 16 * tile + (lane & 15);
  const int64_t row0 = r0 + 16 * half + 4 * (lane >> 4);
  w3.load(a.wf[3], tile, lane);
  float y[4] = {};
  if constexpr (TRAIN) {
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = a.y[min(row0 + r, a.B - 1) * NOUT + col];
  }
  lds_barrier();
  mlp_hidden<2, TRAIN>(a, act[0], act[1], w2, lane, wv, z2);
  const float b = a.bias[NLAYER - 1][col];
  lds_barrier();
  if constexpr (TRAIN) v3.load(a.wb[3], wv, lane);
  mlp_product<1>(act[1], w3, half, lane, &zo);
  if constexpr (!TRAIN) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (a.z_out && row0 + r < a.B) a.z_out[(row0 + r) * NOUT + col] = zo[r] + b;
    if (a.h_last) {
      // whole rows, 8 bytes a lane
      for (int e = t; e < kMlpRows * (HID / 4); e += kMlpThreads) {
        const int r = e / (HID / 4), c = 4 * (e % (HID / 4));
        if (r0 + r < a.B)
          *reinterpret_cast<uint2*>(a.h_last + (r0 + r) * HID + c) = *reinterpret_cast<const uint2*>(&act[1][r][c]);
      }
    }
    return;
  }
  // output gradient 2 (out - y) / (B NOUT), rows beyond the batch zero
  float g[4], lsum = 0.f, sum = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float d = row0 + r < a.B ? (zo[r] + b) - y[r] : 0.f;
    g[r] = 2.f * d / float(a.B * NOUT);
    lsum += d * d;
    sum += g[r];
  }
  const uint2 h = {f2bf2(g[0], g[1]), f2bf2(g[2], g[3])};
  {
    uint16_t(*out)[kActStride] = act[0] + 16 * half + 4 * (lane >> 4);
    out[0][col] = uint16_t(h.x);
    out[1][col] = uint16_t(h.x >> 16);
    out[2][col] = uint16_t(h.y);
    out[3][col] = uint16_t(h.y >> 16);
  }
  reinterpret_cast<uint2*>(a.dfrag[NLAYER - 1])[((int64_t(blockIdx.x) * (NOUT / 16) + tile) * 64 + lane) * 2 + half] = h;
  sum += __shfl_xor(sum, 16);
  sum += __shfl_xor(sum, 32);
  if (half == 1 && lane < 16) bsum[col] = sum;
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) lsum += __shfl_xor(lsum, w);
  if (lane == 0) red[wv] = lsum;
  lds_barrier();
  v2.load(a.wb[2], wv, lane);
  if (half == 0 && lane < 16)
    a.bias_part[int64_t(blockIdx.x) * kBiasCols + bias_col(NLAYER - 1) + col] = sum + bsum[col];
  if (t == 0) {
    float s = 0.f;
    for (int w = 0; w < kMlpThreads / 64; ++w) s += red[w];
    a.loss_part[blockIdx.x] = s;
  }
  mlp_backward_layer<3>(a, act[0], act[1], v3, lane, wv, z2);
  lds_barrier();
  v1.load(a.wb[1], wv, lane);
  mlp_backward_layer<2>(a, act[1], act[0], v2, lane, wv, z1);
  lds_barrier();
  mlp_backward_layer<1>(a, act[0], act[1], v1, lane, wv, z0);
}

// ------------------------------------------------------ weight gradients
// dW = x^T dz of every layer in one launch: a workgroup takes 64 x 64 of one
// layer's gradient (16 x 64 of the first) and one of the `parts` ranges of row
// blocks, its four waves every fourth block, straight from the fragments that
// k_mlp left (they are both operands' own layout: the rows are contracted).
// The waves' sums are added in LDS; the parts in k_params.  The part is the
// fastest index of the grid: consecutive workgroups go to different XCDs, so
// with 8 parts each XCD's L2 reads its own eighth of the fragments.
constexpr int kGradParts = 8;
constexpr int kGradUnits = 4 + 16 + 16 + 8;

__host__ __device__ constexpr int flat_w(int l) {  // layer l's weights in the flat layout
  return l == 0 ? 0 : l == 1 ? 16 * HID + HID : l == 2 ? 16 * HID + HID + HID * HID + HID
                                              : 16 * HID + HID + 2 * (HID * HID + HID);
}
__host__ __device__ constexpr int flat_b(int l) { return flat_w(l) + (l == 0 ? 16 * HID : l < 3 ? HID * HID : HID * NOUT); }
constexpr int kFlat = flat_b(3) + NOUT;

struct GradArgs {
  const uint4* hfrag[NLAYER];
  const uint4* dfrag[NLAYER];
  int64_t blocks;  // of 32 rows
  float* parts;    // [n_parts][kFlat]
  int n_parts;
};

template <int MT>
__device__ __forceinline__ void weight_grad(const GradArgs& a, int part, int l, int m0, int n0, float* lds) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int mts = layer_in(l) / 16, nts = layer_out(l) / 16;
  const int64_t lo = a.blocks * part / a.n_parts, hi = a.blocks * (part + 1) / a.n_parts;
  struct alignas(16) Two { v4s s[2]; };
  const Two* hp = reinterpret_cast<const Two*>(a.hfrag[l]);
  const Two* dp = reinterpret_cast<const Two*>(a.dfrag[l]);
  v4f acc[MT][4];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  Two x[MT], d[4];
  auto load = [&](int64_t blk) {
#pragma unroll
    for (int i = 0; i < MT; ++i) x[i] = hp[(blk * mts + m0 + i) * 64 + lane];
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = dp[(blk * nts + n0 + j) * 64 + lane];
  };
  if (lo + wv < hi) load(lo + wv);
  for (int64_t blk = lo + wv; blk < hi; blk += 4) {
    Two cx[MT], cd[4];
#pragma unroll
    for (int i = 0; i < MT; ++i) cx[i] = x[i];
#pragma unroll
    for (int j = 0; j < 4; ++j) cd[j] = d[j];
    if (blk + 4 < hi) load(blk + 4);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(cx[i].s[h], cd[j].s[h], acc[i][j], 0, 0, 0);
  }
  // element (tile, r, lane) of each wave
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) lds[((wv * MT * 4 + i * 4 + j) * 4 + r) * 64 + lane] = acc[i][j][r];
  __syncthreads();
  float* out = a.parts + int64_t(part) * kFlat + flat_w(l);
  for (int e = t; e < MT * 1024; e += 256) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += lds[w * MT * 1024 + e];
    const int tile = e >> 8, r = (e >> 6) & 3, ln = e & 63;
    const int row = 16 * (m0 + tile / 4) + 4 * (ln >> 4) + r, col = 16 * (n0 + tile % 4) + (ln & 15);
    out[row * layer_out(l) + col] = s;
  }
}

__global__ __launch_bounds__(256) void k_weight_grads(GradArgs a) {
  __shared__ float lds[4 * 4 * 1024];
  const int u = blockIdx.x / a.n_parts, part = blockIdx.x % a.n_parts;
  if (u < 4) weight_grad<1>(a, part, 0, 0, 4 * u, lds);
  else if (u < 36) weight_grad<4>(a, part, 1 + (u - 4) / 16, 4 * ((u - 4) % 16 / 4), 4 * ((u - 4) % 4), lds);
  else weight_grad<4>(a, part, 3, 4 * ((u - 36) / 2), 4 * ((u - 36) % 2), lds);
}

// Sums the parts and either stores the gradient (flat layout) or makes the
// AdamW step, refreshing the bf16 fragments: workgroups 0 .. take 256 weights
// each, then 28 take 32 biases each, then one the loss.
struct ParamArgs {
  const float* parts;
  int n_parts;
  const float* bias_part;
  const float* loss_part;
  int64_t blocks;
  float* grads;   // flat gradient, or NULL: AdamW
  float* loss;    // or NULL
  float *p[NLAYER], *m[NLAYER], *v[NLAYER];     // weights
  float *pb[NLAYER], *mb[NLAYER], *vb[NLAYER];  // biases
  uint16_t *wf[NLAYER], *wb[NLAYER];
  float lr, b1, b2, eps, wd, c1, c2;
};
constexpr int kWeights = kFlat - kBiasCols;
constexpr int kWeightBlocks = kWeights / 256, kBiasBlocks = kBiasCols / 32;
static_assert(kWeights % 256 == 0 && kBiasCols % 32 == 0, "whole workgroups");

__device__ __forceinline__ float adamw(const ParamArgs& a, float* p, float* mm, float* vv, float g, float wd) {
  const float m = a.b1 * *mm + (1.f - a.b1) * g;
  const float v = a.b2 * *vv + (1.f - a.b2) * g * g;
  *mm = m;
  *vv = v;
  float x = *p;
  x -= a.lr * (wd * x + (m * a.c1) / (sqrtf(v * a.c2) + a.eps));
  *p = x;
  return x;
}

__global__ __launch_bounds__(256) void k_params(ParamArgs a) {
  __shared__ float red[256];
  const int t = threadIdx.x, blk = blockIdx.x;
  if (blk < kWeightBlocks) {
    // every layer's weights are whole workgroups
    int e = blk * 256 + t, l = 0;
    while (l < NLAYER - 1 && e >= layer_in(l) * layer_out(l)) e -= layer_in(l) * layer_out(l), ++l;
    float g = 0.f;
#pragma unroll 8
    for (int p = 0; p < a.n_parts; ++p) g += a.parts[int64_t(p) * kFlat + flat_w(l) + e];
    if (a.grads) {
      a.grads[flat_w(l) + e] = g;
      return;
    }
    const uint16_t h = f2bf(adamw(a, a.p[l] + e, a.m[l] + e, a.v[l] + e, g, a.wd));
    const int k = e / layer_out(l), n = e % layer_out(l);
    a.wf[l][frag_fwd(layer_in(l), k, n)] = h;
    if (l > 0) a.wb[l][frag_bwd(layer_out(l), k, n)] = h;
  } else if (blk < kWeightBlocks + kBiasBlocks) {
    const int c = 32 * (blk - kWeightBlocks) + (t & 31), j = t >> 5;
    float s = 0.f;
#pragma unroll 8
    for (int64_t b = j; b < a.blocks; b += 8) s += a.bias_part[b * kBiasCols + c];
    red[t] = s;
    __syncthreads();
    if (t >= 32) return;
#pragma unroll
    for (int i = 1; i < 8; ++i) s += red[32 * i + t];
    const int l = min(c / HID, NLAYER - 1), o = c - bias_col(l);
    if (a.grads) a.grads[flat_b(l) + o] = s;
    else adamw(a, a.pb[l] + o, a.mb[l] + o, a.vb[l] + o, s, 0.f);  // biases are not decayed
  } else {
    float s = 0.f;
    for (int64_t b = t; b < a.blocks; b += 256) s += a.loss_part[b];
    red[t] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (t < w) red[t] += red[t + w];
      __syncthreads();
    }
    if (t == 0) a.loss[0] = red[0];
  }
}

// bf16 fragments of layer l's weights W [nin][nout]
__global__ __launch_bounds__(256) void k_weights_bf16(const float* W, int nin, int nout, uint16_t* wf, uint16_t* wb) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= nin * nout) return;
  const uint16_t h = f2bf(W[e]);
  wf[frag_fwd(nin, e / nout, e % nout)] = h;
  if (nin > 16) wb[frag_bwd(nout, e / nout, e % nout)] = h;
}

__global__ void k_bf16_to_f32(const uint16_t* x, int64_t n, float* y) {
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e < n) y[e] = bf2f(x[e]);
}

// --------------------------------------------------------- reconstruction
// coefficients = phi A + zstd * z + zmean; node values = mean + coef V;
// also the predicted log10 mismatch from the last hidden layer.
struct ReconArgs {
  const double* params;  // [12][pB], columns b0 ..
  int64_t pB, b0;
  const float* z;        // [B][NOUT]
  const float* A;        // [NFEAT][NOUT]
  const float* zmean;
  const float* zstd;
  const float* basis;    // [2][NBAS][NN]
  const double* mean;    // [2][NN]
  const uint16_t* h3;    // [B][HID] last hidden layer (bf16)
  const float* head;     // [HID + 1]
  int64_t B;
  float* nodes;          // [B][2][NN]
  float* logmm;          // [B] or NULL
};

// per sample: skip-path features phi (the PN coefficients times 3/(128 eta)),
// coefficients and predicted log10 mismatch
__global__ __launch_bounds__(256) void k_coefficients(ReconArgs a, float* coef) {
  __shared__ float red[256];
  const int64_t b = blockIdx.x;
  const int t = threadIdx.x;
  if (t < NOUT) {
    const double* p = a.params + a.b0 + b;
    const double q = p[a.pB], chi1 = p[2 * a.pB], chi2 = p[3 * a.pB];
    const double eta = q / ((1.0 + q) * (1.0 + q));
    double c[8], lg[8];
    pn_coefficients(eta, q, chi1, chi2, c, lg);
    const double pre = 3.0 / (128.0 * eta);
    const double f[NFEAT] = {pre * c[2], pre * c[3], pre * c[4], pre * c[5], pre * c[6], pre * c[7], pre * lg[5],
                             pre * lg[6], 1.0};
    double s = 0.0;
#pragma unroll
    for (int fi = 0; fi < NFEAT; ++fi) s += f[fi] * double(a.A[fi * NOUT + t]);
    coef[b * NOUT + t] = float(s + double(a.zstd[t]) * double(a.z[b * NOUT + t]) + double(a.zmean[t]));
  }
  if (!a.logmm) return;
  red[t] = (t < HID) ? bf2f(a.h3[b * HID + t]) * a.head[t] : 0.f;
  for (int w = 128; w > 0; w >>= 1) {
    __syncthreads();
    if (t < w) red[t] += red[t + w];
  }
  if (t == 0) a.logmm[b] = red[0] + a.head[HID];
}

// nodes[b][part][j] = mean[part][j] + sum_k coef[b][part*64 + k] V[part][k][j]
// on the matrix cores (binary32, 16x16x4): 32 samples by 64 nodes per wave,
// grid (NN/256, ceil(B/32), 2).  Lane c + 16 g supplies k = 16 g + s in step s,
// so that it reads a sample's coefficients as four 16-byte loads.
__global__ __launch_bounds__(256) void k_reconstruct(ReconArgs a, const float* coef) {
  const int part = blockIdx.z, t = threadIdx.x, lane = t & 63, c = lane & 15, g = lane >> 4;
  const int64_t b0 = int64_t(blockIdx.y) * 32;
  const int j0 = blockIdx.x * 256 + (t >> 6) * 64;
  const float* V = a.basis + (size_t(part) * NBAS + 16 * g) * NN + j0 + c;
  float ca[2][16];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t b = min(b0 + 16 * i + c, a.B - 1);  // rows beyond the batch repeat its last and are not stored
    const float4* p = reinterpret_cast<const float4*>(coef + b * NOUT + part * NBAS + 16 * g);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = p[q];
      ca[i][4 * q] = v.x;
      ca[i][4 * q + 1] = v.y;
      ca[i][4 * q + 2] = v.z;
      ca[i][4 * q + 3] = v.w;
    }
  }
  v4f acc[2][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float m = float(a.mean[part * NN + j0 + 16 * j + c]);
    acc[0][j] = acc[1][j] = v4f{m, m, m, m};
  }
#pragma unroll
  for (int s = 0; s < 16; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float v = V[size_t(s) * NN + 16 * j];
      acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[0][s], v, acc[0][j], 0, 0, 0);
      acc[1][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[1][s], v, acc[1][j], 0, 0, 0);
    }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t b = b0 + 16 * i + 4 * g + r;
      if (b < a.B)
#pragma unroll
        for (int j = 0; j < 4; ++j) a.nodes[(b * 2 + part) * NN + j0 + 16 * j + c] = acc[i][j][r];
    }
}

// h+, hx on the window grid from node values (binary64 Newtonian phase,
// binary32 interpolated residual, hardware sine/cosine on the reduced phase)
struct SurrWaveArgs {
  DevCfg cf;
  const double* params;
  int64_t B;
  const float* nodes;   // [B][2][NN]
  const double* k53;    // [F] k^(-5/3)
  const double* lnk3;   // [F] ln(k)/3
  float* hp;
  float* hc;
};

__device__ __forceinline__ float node_interp(const float* v, float u) {
  u = fminf(fmaxf(u, 0.f), float(NN - 1));
  int i = min(int(u), NN - 2);
  const float t = u - float(i);
  return (1.f - t) * v[i] + t * v[i + 1];
}

__global__ __launch_bounds__(256) void k_surrogate_waveform(SurrWaveArgs a) {
  __shared__ double sh[8];
  const int64_t b = blockIdx.x;
  const int64_t B = a.B;
  if (threadIdx.x == 0) {
    const double mc = a.params[0 * B + b], q = a.params[1 * B + b];
    const double eta = q / ((1.0 + q) * (1.0 + q));
    const double Ms = mc * pow(eta, -0.6) * kMsunSec;
    sh[0] = Ms;
    const double v1 = cbrt(kPi * Ms * a.cf.invT);
    // Newtonian phase 3/(128 eta v^5) in revolutions at bin k: sh[1] k^(-5/3)
    sh[1] = 3.0 / (128.0 * eta) / (2.0 * kPi) / (v1 * v1 * v1 * v1 * v1);
    sh[2] = v1;
    sh[3] = (-a.params[9 * B + b] - 0.25 * kPi) / (2.0 * kPi);         // pconst
    const double A0 = kStrainScale * sqrt(5.0 / 24.0) * pow(kPi, -2.0 / 3.0) *
                      pow(mc * kMsunSec, 5.0 / 6.0) / (a.params[4 * B + b] * kMpcSec);
    sh[4] = A0 * pow(a.cf.T, 7.0 / 6.0);
    sh[5] = cos(a.params[5 * B + b]);
    sh[6] = 0.2 / Ms;                                                   // f_cut
    sh[7] = (log(Ms * a.cf.invT) - log(MF_LO)) / (log(MF_HI / MF_LO) / double(NN - 1));
  }
  __syncthreads();
  const int F = a.cf.F;
  const float* nr = a.nodes + (b * 2 + 0) * NN;
  const float* np_ = a.nodes + (b * 2 + 1) * NN;
  const double inv_dlog = double(NN - 1) / log(MF_HI / MF_LO);
  for (int k = threadIdx.x; k < F; k += 256) {
    float2 hp = {0.f, 0.f}, hc = {0.f, 0.f};
    const double f = double(k) * a.cf.invT;
    if (k > 0 && k >= a.cf.kmin && f < sh[6] && k < a.cf.N / 2) {
      // ln k = 3 * (ln(k)/3) from the table
      const float u = float(sh[7] + 3.0 * a.lnk3[k] * inv_dlog);
      const float ratio = node_interp(nr, u);
      const float dpsi = node_interp(np_, u);
      const double k53 = a.k53[k];
      double rev = sh[1] * k53 + double(dpsi) * (1.0 / (2.0 * kPi)) + sh[3];
      rev = frac1(rev);
      float s, c;
      sincos_rev(float(rev), &s, &c);
      // A_N = A0T k^(-7/6) = A0T k^(-5/3) k^(1/2)
      const float kf = float(k);
      const float A = float(sh[4]) * float(k53) * (kf * rsqrt_t(kf)) * ratio;
      const float cp = A * 0.5f * (1.f + float(sh[5] * sh[5]));
      const float cx = A * float(sh[5]);
      hp = {cp * c, -cp * s};
      hc = {-cx * s, -cx * c};
    }
    reinterpret_cast<float2*>(a.hp)[b * F + k] = hp;
    reinterpret_cast<float2*>(a.hc)[b * F + k] = hc;
  }
}

// ---------------------------------------------------------------- mismatch
// <a|b> = 4 df Re sum a conj(b) / S over kept bins; binary64 accumulation.
struct MismatchArgs {
  const float* ha; const float* hb;  // [B][F] complex
  const float* psd;                  // [F] one-sided PSD on the window grid
  int64_t B; int F; int kmin; double df;
  const double* params;              // for f_cut (IMR-form), may be NULL
  double* mm;
};
__global__ __launch_bounds__(256) void k_mismatch(MismatchArgs a) {
  __shared__ double r0[256], r1[256], r2[256];
  const int64_t b = blockIdx.x;
  const int t = threadIdx.x;
  double kcut = double(a.F - 1);
  if (a.params) {
    const double mc = a.params[b], q = a.params[a.B + b];
    const double eta = q / ((1.0 + q) * (1.0 + q));
    kcut = (0.2 / (mc * pow(eta, -0.6) * kMsunSec)) / a.df;
  }
  double s0 = 0, s1 = 0, s2 = 0;
  const float2* A = reinterpret_cast<const float2*>(a.ha) + b * a.F;
  const float2* Bv = reinterpret_cast<const float2*>(a.hb) + b * a.F;
  for (int k = max(a.kmin, 1) + t; k < a.F - 1; k += 256) {
    if (double(k) >= kcut) continue;
    const double w = 1.0 / double(a.psd[k]);
    const float2 x = A[k], y = Bv[k];
    s0 += (double(x.x) * y.x + double(x.y) * y.y) * w;
    s1 += (double(x.x) * x.x + double(x.y) * x.y) * w;
    s2 += (double(y.x) * y.x + double(y.y) * y.y) * w;
  }
  r0[t] = s0; r1[t] = s1; r2[t] = s2;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) { r0[t] += r0[t + w]; r1[t] += r1[t + w]; r2[t] += r2[t + w]; }
    __syncthreads();
  }
  if (t == 0) {
    const double aa = r1[0], bb = r2[0];
    a.mm[b] = (aa > 0.0 && bb > 0.0) ? 1.0 - r0[0] / sqrt(aa * bb) : 0.0;
  }
}

// Mismatch maximised over a time shift and a phase offset of hb.  With
// z_k = a_k conj(b_k) / S_k on the kept bins (all below NC = N/2), the overlap
// of a with b delayed by s T / NC and rotated by phi is Re(e^{i phi} c(s)),
// c(s) = sum_k z_k e^{2 pi i k s / NC}; its maximum over phi is |c(s)|.  One
// inverse transform gives c on the NC integer shifts; around the best of them
// |c| is evaluated directly (binary64 sums) at s - 1, s, s + 1; each further
// stage centres three points, a quarter and then a sixteenth of a step apart,
// on the previous parabola's vertex, and the last vertex is evaluated too; the
// largest value evaluated is the maximum.  One workgroup of NC/16 threads per
// pair.
struct MismatchMaxArgs {
  const float* ha; const float* hb;  // [B][F] complex
  const float* psd;                  // [F]
  int64_t B; int F; int kmin; double df;
  const double* params;              // for f_cut (IMR-form), may be NULL
  const cpx<float>* tw;              // pass twiddle tables of the NC-point transform
  double* mm;
};

template <int NC>
__global__ __launch_bounds__(NC / 16) void k_mismatch_max(MismatchMaxArgs a) {
  constexpr int NT = NC / 16, LS = LdsSize<NC>::value;
  __shared__ float lds[2 * LS];
  const int t = threadIdx.x;
  const int64_t b = blockIdx.x;
  double kcut = double(a.F - 1);
  if (a.params) {
    const double mc = a.params[b], q = a.params[a.B + b];
    const double eta = q / ((1.0 + q) * (1.0 + q));
    kcut = (0.2 / (mc * pow(eta, -0.6) * kMsunSec)) / a.df;
  }
  const float2* A = reinterpret_cast<const float2*>(a.ha) + b * a.F;
  const float2* Bv = reinterpret_cast<const float2*>(a.hb) + b * a.F;
  // z_k for this thread's bins k = t + NT j (all below NC = F - 1); built
  // before the transform and again after it, so that it is not kept live
  // through the transform
  double aa = 0.0, bb = 0.0;
  auto zk = [&](int j, bool norms) {
    const int k = t + NT * j;
    cpx<float> z = {0.f, 0.f};
    if (k >= max(a.kmin, 1) && k < a.F - 1 && double(k) < kcut) {
      const double w = 1.0 / double(a.psd[k]);
      const float2 x = A[k], y = Bv[k];
      z = {float((double(x.x) * y.x + double(x.y) * y.y) * w), float((double(x.y) * y.x - double(x.x) * y.y) * w)};
      if (norms) {
        aa += (double(x.x) * x.x + double(x.y) * x.y) * w;
        bb += (double(y.x) * y.x + double(y.y) * y.y) * w;
      }
    }
    return z;
  };
  cpx<float> v[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) v[fft_in_slot<NC, 0>(j)] = zk(j, true);
  double* red = reinterpret_cast<double*>(lds);  // 2 NT doubles, while the planes are idle
  auto reduce2 = [&](double u, double v2, double& ru, double& rv) {
    __syncthreads();
    red[t] = u;
    red[NT + t] = v2;
    __syncthreads();
    for (int w = NT / 2; w > 0; w >>= 1) {
      if (t < w) {
        red[t] += red[t + w];
        red[NT + t] += red[NT + t + w];
      }
      __syncthreads();
    }
    ru = red[0];
    rv = red[NT];
  };
  double AA, BB;
  reduce2(aa, bb, AA, BB);
  cpx<float> z[16];  // filled after the transform
  // |c(s)| summed directly in binary64 (phases reduced in binary64 first)
  auto cabs_at = [&](double s) {
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int k = t + NT * j;
      const double rev = frac1(double(k) * s * (1.0 / double(NC)));
      float sn, cs;
      sincos_rev(float(rev), &sn, &cs);
      re += double(z[j].x) * cs - double(z[j].y) * sn;
      im += double(z[j].x) * sn + double(z[j].y) * cs;
    }
    double R, I;
    reduce2(re, im, R, I);
    return sqrt(R * R + I * I);
  };
  // coarse maximum over the NC integer shifts
  __syncthreads();
  block_fft<float, NC, +1, false, 0>(v, lds, lds + LS, t, PassTwiddle<float, NC, 0>{a.tw});
  float best = -1.f;
  int bi = 0;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const float m2 = v[e].x * v[e].x + v[e].y * v[e].y;
    const int n = fft_out_index<NC, 0>(t, e);
    if (m2 > best || (m2 == best && n < bi)) { best = m2; bi = n; }
  }
  __syncthreads();  // the transform's last reads are done: the planes become scratch
  float* fv = lds;
  int* fi = reinterpret_cast<int*>(lds + NT);
  fv[t] = best;
  fi[t] = bi;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (t < w) {
      const float o = fv[t + w];
      const int oi = fi[t + w];
      if (o > fv[t] || (o == fv[t] && oi < fi[t])) { fv[t] = o; fi[t] = oi; }
    }
    __syncthreads();
  }
  const double s0 = double(fi[0]);
#pragma unroll
  for (int j = 0; j < 16; ++j) z[j] = zk(j, false);
  // parabolic refinement on directly summed values
  auto vertex = [](double h, double gm, double g0, double gp) {
    const double den = gm - 2.0 * g0 + gp;
    if (!(den < 0.0)) return 0.0;  // not a maximum: stay
    const double x = 0.5 * h * (gm - gp) / den;
    return fmin(fmax(x, -h), h);
  };
  const double gm = cabs_at(s0 - 1.0), g0 = cabs_at(s0), gp = cabs_at(s0 + 1.0);
  const double s1 = s0 + vertex(1.0, gm, g0, gp);
  const double h1 = 0.25;
  const double g1m = cabs_at(s1 - h1), g1 = cabs_at(s1), g1p = cabs_at(s1 + h1);
  const double s2 = s1 + vertex(h1, g1m, g1, g1p);
  const double h2 = 0.0625;
  const double g2m = cabs_at(s2 - h2), g2 = cabs_at(s2), g2p = cabs_at(s2 + h2);
  const double g3 = cabs_at(s2 + vertex(h2, g2m, g2, g2p));
  const double c0 = cabs_at(0.0);  // the strict alignment is always a candidate
  const double gmax = fmax(fmax(fmax(fmax(g0, gm), fmax(gp, g1)), fmax(fmax(g1m, g1p), fmax(g2m, g2))),
                           fmax(fmax(g2p, g3), c0));
  if (t == 0) a.mm[b] = (AA > 0.0 && BB > 0.0) ? 1.0 - gmax / sqrt(AA * BB) : 0.0;
}

}  // namespace

// ======================================================================= host

struct gw_surrogate {
  gw_ctx* ctx = nullptr;
  float lo[4], hi[4];
  float* basis = nullptr;   // [2][NBAS][NN]
  double* mean = nullptr;   // [2][NN]
  float* A = nullptr;       // [NFEAT][NOUT]
  float* zmean = nullptr;   // [NOUT]
  float* zstd = nullptr;    // [NOUT]
  float* head = nullptr;    // [HID + 1]
  float* W[NLAYER] = {};
  float* b[NLAYER] = {};
  uint16_t* wf[NLAYER] = {};    // bf16 fragments of the weights, forward order
  uint16_t* wb[NLAYER] = {};    // and backward order (layers 1..)
  float* mW[NLAYER] = {};
  float* vW[NLAYER] = {};
  float* mb[NLAYER] = {};
  float* vb[NLAYER] = {};
  int64_t step = 0;
  double beta1 = 0.9, beta2 = 0.999, eps = 1e-8;  // AdamW hyper-parameters
  int64_t bmax = 0;
  // scratch for bmax rows (bblk = ceil(bmax/32) blocks of 32)
  uint4* hfrag[NLAYER] = {};    // [bblk][in/16][64]
  uint4* dfrag[NLAYER] = {};    // [bblk][out/16][64]
  float* bias_part = nullptr;   // [bblk][kBiasCols]
  float* loss_part = nullptr;   // [bblk]
  float* parts = nullptr;       // [kGradParts][kFlat]
  float* zout = nullptr;        // [bmax][NOUT] output layer
  uint16_t* hlast = nullptr;    // [bmax][HID] last hidden layer
  float* coef = nullptr;        // [bmax][NOUT]
  std::string err;
};

namespace {

gw_status sfail(gw_surrogate* s, gw_status st, const std::string& m) {
  if (s) s->err = m;
  return st;
}
gw_status slaunch(gw_surrogate* s, const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return sfail(s, GW_EHIP, std::string(what) + ": " + hipGetErrorString(e));
  return GW_OK;
}
unsigned nblk(int64_t n) { return unsigned((n + 255) / 256); }

template <class T> bool dalloc(T** p, size_t n) { return hipMalloc(reinterpret_cast<void**>(p), sizeof(T) * n) == hipSuccess; }

MlpArgs mlp_args(const gw_surrogate* s, const float* theta, int64_t B) {
  MlpArgs a{};
  a.theta = theta;
  a.B = B;
  for (int c = 0; c < 4; ++c) { a.lo[c] = s->lo[c]; a.hi[c] = s->hi[c]; }
  for (int l = 0; l < NLAYER; ++l) {
    a.wf[l] = s->wf[l];
    a.wb[l] = s->wb[l];
    a.bias[l] = s->b[l];
  }
  return a;
}

unsigned mlp_blocks(int64_t B) { return unsigned((B + kMlpRows - 1) / kMlpRows); }

// output layer to z_out, last hidden layer to h_last (either may be NULL)
gw_status mlp_infer(gw_surrogate* s, MlpArgs a, float* z_out, uint16_t* h_last, hipStream_t st) {
  a.z_out = z_out;
  a.h_last = h_last;
  hipLaunchKernelGGL((k_mlp<false>), dim3(mlp_blocks(a.B)), dim3(kMlpThreads), 0, st, a);
  return slaunch(s, "mlp inference");
}

// Forward and backward pass, then the gradients (flat layout) or, with grads
// NULL, the AdamW step of `u`.  Three launches: 37 of layer-by-layer products,
// sums and element-wise passes took 258 us at 8192 rows, of which the products'
// arithmetic is 7 us at the rate of a large matrix product.
gw_status mlp_train(gw_surrogate* s, const float* theta, const float* z, int64_t B, float* grads, float* loss, ParamArgs u,
                    hipStream_t st) {
  MlpArgs a = mlp_args(s, theta, B);
  a.y = z;
  GradArgs g{};
  for (int l = 0; l < NLAYER; ++l) {
    g.hfrag[l] = a.hfrag[l] = s->hfrag[l];
    g.dfrag[l] = a.dfrag[l] = s->dfrag[l];
  }
  a.bias_part = s->bias_part;
  a.loss_part = s->loss_part;
  const unsigned blocks = mlp_blocks(B);
  hipLaunchKernelGGL((k_mlp<true>), dim3(blocks), dim3(kMlpThreads), 0, st, a);
  gw_status r = slaunch(s, "mlp forward and backward");
  if (r != GW_OK) return r;
  g.blocks = blocks;
  g.parts = s->parts;
  // a wave of a part takes every fourth of its blocks
  const int parts = int(std::min<int64_t>(kGradParts, (blocks + 3) / 4));
  g.n_parts = parts;
  hipLaunchKernelGGL(k_weight_grads, dim3(unsigned(kGradUnits * parts)), dim3(256), 0, st, g);
  r = slaunch(s, "weight gradients");
  if (r != GW_OK) return r;
  u.parts = s->parts;
  u.n_parts = parts;
  u.bias_part = s->bias_part;
  u.loss_part = s->loss_part;
  u.blocks = blocks;
  u.grads = grads;
  u.loss = loss;
  for (int l = 0; l < NLAYER; ++l) {
    u.p[l] = s->W[l];
    u.m[l] = s->mW[l];
    u.v[l] = s->vW[l];
    u.pb[l] = s->b[l];
    u.mb[l] = s->mb[l];
    u.vb[l] = s->vb[l];
    u.wf[l] = s->wf[l];
    u.wb[l] = s->wb[l];
  }
  hipLaunchKernelGGL(k_params, dim3(unsigned(kWeightBlocks + kBiasBlocks + (loss ? 1 : 0))), dim3(256), 0, st, u);
  return slaunch(s, "parameter update");
}

int64_t layer_wn(int l) { return int64_t(layer_in(l)) * layer_out(l); }
int64_t n_weights_flat() {
  int64_t n = 0;
  for (int l = 0; l < NLAYER; ++l) n += layer_wn(l) + layer_out(l);
  return n;
}

}  // namespace

extern "C" {

gw_status gw_surrogate_destroy(gw_surrogate* s) {
  if (!s) return GW_OK;
  void* ptrs[] = {s->basis, s->mean, s->A, s->zmean, s->zstd, s->head, s->bias_part, s->loss_part, s->parts,
                  s->zout, s->hlast, s->coef};
  for (void* p : ptrs) (void)hipFree(p);
  for (int l = 0; l < NLAYER; ++l) {
    void* q[] = {s->W[l], s->b[l], s->wf[l], s->wb[l], s->mW[l], s->vW[l], s->mb[l], s->vb[l], s->hfrag[l], s->dfrag[l]};
    for (void* p : q) (void)hipFree(p);
  }
  delete s;
  return GW_OK;
}

gw_status gw_surrogate_create(gw_ctx* ctx, int64_t max_batch, gw_surrogate** out) {
  if (!ctx || !out || max_batch < 1 || max_batch > (int64_t(1) << 20)) return GW_EINVAL;
  *out = nullptr;
  if (ctx->dc.approximant != 1) return gw::ctx_fail(ctx, GW_EUNSUPPORTED, "the surrogate models approximant 1");
  gw_surrogate* s = new gw_surrogate();
  s->ctx = ctx;
  const gw_config& c = ctx->cfg;
  s->lo[0] = float(c.mc[0]); s->hi[0] = float(c.mc[1]);
  s->lo[1] = float(c.q[0]); s->hi[1] = float(c.q[1]);
  s->lo[2] = s->lo[3] = float(c.chi[0]);
  s->hi[2] = s->hi[3] = float(c.chi[1]);
  for (int i = 0; i < 4; ++i)
    if (!(s->hi[i] > s->lo[i])) s->hi[i] = s->lo[i] + 1.0f;
  s->bmax = max_batch;
  const int64_t B = max_batch, blocks = mlp_blocks(max_batch);
  bool ok = dalloc(&s->basis, 2 * NBAS * NN) && dalloc(&s->mean, 2 * NN) && dalloc(&s->A, NFEAT * NOUT) &&
            dalloc(&s->zmean, NOUT) && dalloc(&s->zstd, NOUT) && dalloc(&s->head, HID + 1) &&
            dalloc(&s->bias_part, size_t(blocks) * kBiasCols) && dalloc(&s->loss_part, size_t(blocks)) &&
            dalloc(&s->parts, size_t(kGradParts) * kFlat) && dalloc(&s->zout, B * NOUT) && dalloc(&s->hlast, B * HID) &&
            dalloc(&s->coef, B * NOUT);
  for (int l = 0; l < NLAYER && ok; ++l) {
    const int64_t wn = layer_wn(l), bo = layer_out(l);
    ok = dalloc(&s->W[l], wn) && dalloc(&s->b[l], bo) && dalloc(&s->wf[l], wn) && dalloc(&s->wb[l], wn) && dalloc(&s->mW[l], wn) &&
         dalloc(&s->vW[l], wn) && dalloc(&s->mb[l], bo) && dalloc(&s->vb[l], bo) &&
         dalloc(&s->hfrag[l], size_t(blocks) * (layer_in(l) / 16) * 64) && dalloc(&s->dfrag[l], size_t(blocks) * (bo / 16) * 64);
  }
  if (!ok) {
    gw_surrogate_destroy(s);
    return GW_ENOMEM;
  }
  // zero the state; weights are set by gw_surrogate_set_weights
  std::vector<float> zeros(size_t(std::max<int64_t>(HID * HID, 2 * NBAS * NN)), 0.f);
  std::vector<float> ones(NOUT, 1.f);
  auto up = [&](void* dst, const void* src, size_t bytes) {
    return ok && (ok = hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice) == hipSuccess);
  };
  ok = true;
  up(s->head, zeros.data(), sizeof(float) * (HID + 1));
  up(s->zmean, zeros.data(), sizeof(float) * NOUT);
  up(s->zstd, ones.data(), sizeof(float) * NOUT);
  up(s->A, zeros.data(), sizeof(float) * NFEAT * NOUT);
  for (int l = 0; l < NLAYER; ++l) {
    const int64_t wn = layer_wn(l), bo = layer_out(l);
    up(s->W[l], zeros.data(), sizeof(float) * wn);
    up(s->b[l], zeros.data(), sizeof(float) * bo);
    up(s->mW[l], zeros.data(), sizeof(float) * wn);
    up(s->vW[l], zeros.data(), sizeof(float) * wn);
    up(s->mb[l], zeros.data(), sizeof(float) * bo);
    up(s->vb[l], zeros.data(), sizeof(float) * bo);
    up(s->wf[l], zeros.data(), sizeof(uint16_t) * wn);
    up(s->wb[l], zeros.data(), sizeof(uint16_t) * wn);
  }
  if (!ok || hipDeviceSynchronize() != hipSuccess) {
    gw_surrogate_destroy(s);
    return GW_EHIP;
  }
  *out = s;
  return GW_OK;
}

const char* gw_surrogate_last_error(const gw_surrogate* s) { return s ? s->err.c_str() : "surrogate is NULL"; }

int64_t gw_surrogate_n_weights(void) { return n_weights_flat(); }

gw_status gw_surrogate_set_weights(gw_surrogate* s, const float* host_flat, int64_t n) {
  if (!s || !host_flat || n != n_weights_flat()) return GW_EINVAL;
  const float* p = host_flat;
  for (int l = 0; l < NLAYER; ++l) {
    const int64_t wn = layer_wn(l), bo = layer_out(l);
    if (hipMemcpy(s->W[l], p, sizeof(float) * wn, hipMemcpyHostToDevice) != hipSuccess) return GW_EHIP;
    p += wn;
    if (hipMemcpy(s->b[l], p, sizeof(float) * bo, hipMemcpyHostToDevice) != hipSuccess) return GW_EHIP;
    p += bo;
    hipLaunchKernelGGL(k_weights_bf16, dim3(nblk(wn)), dim3(256), 0, 0, s->W[l], layer_in(l), layer_out(l), s->wf[l],
                       s->wb[l]);
  }
  s->step = 0;
  for (int l = 0; l < NLAYER; ++l) {
    if (hipMemset(s->mW[l], 0, sizeof(float) * layer_wn(l)) != hipSuccess ||
        hipMemset(s->vW[l], 0, sizeof(float) * layer_wn(l)) != hipSuccess ||
        hipMemset(s->mb[l], 0, sizeof(float) * layer_out(l)) != hipSuccess ||
        hipMemset(s->vb[l], 0, sizeof(float) * layer_out(l)) != hipSuccess)
      return sfail(s, GW_EHIP, "set_weights: moment reset");
  }
  if (hipDeviceSynchronize() != hipSuccess) return sfail(s, GW_EHIP, "set_weights");
  return GW_OK;
}

gw_status gw_surrogate_get_weights(gw_surrogate* s, float* host_flat, int64_t n) {
  if (!s || !host_flat || n != n_weights_flat()) return GW_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return sfail(s, GW_EHIP, "get_weights");
  float* p = host_flat;
  for (int l = 0; l < NLAYER; ++l) {
    const int64_t wn = layer_wn(l), bo = layer_out(l);
    if (hipMemcpy(p, s->W[l], sizeof(float) * wn, hipMemcpyDeviceToHost) != hipSuccess) return GW_EHIP;
    p += wn;
    if (hipMemcpy(p, s->b[l], sizeof(float) * bo, hipMemcpyDeviceToHost) != hipSuccess) return GW_EHIP;
    p += bo;
  }
  return GW_OK;
}

gw_status gw_surrogate_targets(gw_surrogate* s, const double* params, int64_t B, float* ratio, float* dpsi,
                               double* feat, hipStream_t st) {
  if (!s || B < 0 || B > 0x7fffffff) return GW_EINVAL;
  if (B == 0) return GW_OK;
  if (!params || !ratio || !dpsi || !feat) return sfail(s, GW_EINVAL, "NULL pointer");
  TargetArgs a{s->ctx->dc, params, B, ratio, dpsi, feat};
  hipLaunchKernelGGL(k_targets, dim3(unsigned(B)), dim3(256), 0, st, a);
  return slaunch(s, "k_targets");
}

// Basis of each target set from its first n rows (synchronous: the
// eigen-decomposition of the 1024 x 1024 Gram matrices runs on the host).
gw_status gw_surrogate_fit_basis(gw_surrogate* s, const float* ratio, const float* dpsi, int64_t n, hipStream_t st) {
  if (!s || !ratio || !dpsi || n < NBAS) return GW_EINVAL;
  double* G = nullptr;
  if (!dalloc(&G, size_t(NN) * NN)) return sfail(s, GW_ENOMEM, "Gram buffer");
  std::vector<double> hG(size_t(NN) * NN), w;
  std::vector<float> hb(size_t(NBAS) * NN);
  for (int part = 0; part < 2; ++part) {
    const float* X = part == 0 ? ratio : dpsi;
    hipLaunchKernelGGL(k_colmean, dim3(NN / 256), dim3(256), 0, st, X, n, s->mean + part * NN);
    hipLaunchKernelGGL(k_gram, dim3(NN / 32, NN / 32), dim3(256), 0, st, X, n, s->mean + part * NN, G);
    if (hipStreamSynchronize(st) != hipSuccess ||
        hipMemcpy(hG.data(), G, sizeof(double) * NN * NN, hipMemcpyDeviceToHost) != hipSuccess) {
      (void)hipFree(G);
      return sfail(s, GW_EHIP, "Gram");
    }
    sym_eig(hG, NN, w);
    std::vector<int> idx(NN);
    for (int i = 0; i < NN; ++i) idx[i] = i;
    std::sort(idx.begin(), idx.end(), [&](int x, int y) { return w[x] > w[y]; });
    for (int k = 0; k < NBAS; ++k) {
      const int col = idx[k];
      // sign: largest-magnitude component positive
      double big = 0.0;
      for (int j = 0; j < NN; ++j)
        if (std::fabs(hG[size_t(col) * NN + j]) > std::fabs(big)) big = hG[size_t(col) * NN + j];
      const double sg = big < 0 ? -1.0 : 1.0;
      for (int j = 0; j < NN; ++j) hb[size_t(k) * NN + j] = float(sg * hG[size_t(col) * NN + j]);
    }
    if (hipMemcpy(s->basis + size_t(part) * NBAS * NN, hb.data(), sizeof(float) * NBAS * NN, hipMemcpyHostToDevice) !=
        hipSuccess) {
      (void)hipFree(G);
      return sfail(s, GW_EHIP, "basis upload");
    }
  }
  (void)hipFree(G);
  return GW_OK;
}

gw_status gw_surrogate_project(gw_surrogate* s, const float* ratio, const float* dpsi, int64_t n, float* C, hipStream_t st) {
  if (!s || !ratio || !dpsi || !C || n < 0) return GW_EINVAL;
  if (n == 0) return GW_OK;
  const unsigned g = unsigned((n + 63) / 64);
  hipLaunchKernelGGL(k_project_basis, dim3(g), dim3(256), 0, st, ratio, n, s->mean, s->basis, C, NOUT, 0);
  hipLaunchKernelGGL(k_project_basis, dim3(g), dim3(256), 0, st, dpsi, n, s->mean + NN, s->basis + NBAS * NN, C, NOUT, NBAS);
  return slaunch(s, "k_project_basis");
}

// Skip path by least squares and standardisation of the residual
// (synchronous).  Z receives the standardised residual targets [n][NOUT].
gw_status gw_surrogate_fit_skip(gw_surrogate* s, const double* feat, const float* C, int64_t n, float* Z, hipStream_t st) {
  if (!s || !feat || !C || !Z || n < NFEAT) return GW_EINVAL;
  double *P = nullptr, *Q = nullptr;
  if (!dalloc(&P, NFEAT * NFEAT) || !dalloc(&Q, NFEAT * NOUT)) return sfail(s, GW_ENOMEM, "normal equations");
  hipLaunchKernelGGL(k_normal_eq, dim3(NOUT + NFEAT), dim3(256), 0, st, feat, C, n, P, Q);
  std::vector<double> hP(NFEAT * NFEAT), hQ(NFEAT * NOUT);
  if (hipStreamSynchronize(st) != hipSuccess || hipMemcpy(hP.data(), P, sizeof(double) * NFEAT * NFEAT, hipMemcpyDeviceToHost) != hipSuccess ||
      hipMemcpy(hQ.data(), Q, sizeof(double) * NFEAT * NOUT, hipMemcpyDeviceToHost) != hipSuccess) {
    (void)hipFree(P); (void)hipFree(Q);
    return sfail(s, GW_EHIP, "normal equations");
  }
  (void)hipFree(P); (void)hipFree(Q);
  // scale columns for conditioning
  std::vector<double> sc(NFEAT);
  for (int i = 0; i < NFEAT; ++i) sc[i] = 1.0 / std::sqrt(std::max(hP[i * NFEAT + i], 1e-300));
  for (int i = 0; i < NFEAT; ++i) {
    for (int j = 0; j < NFEAT; ++j) hP[i * NFEAT + j] *= sc[i] * sc[j];
    hP[i * NFEAT + i] *= 1.0 + 1e-12;
    for (int c = 0; c < NOUT; ++c) hQ[i * NOUT + c] *= sc[i];
  }
  if (!chol_solve(hP, NFEAT, hQ, NOUT)) return sfail(s, GW_EINVAL, "skip path: singular normal equations");
  std::vector<float> hA(NFEAT * NOUT);
  for (int i = 0; i < NFEAT; ++i)
    for (int c = 0; c < NOUT; ++c) hA[i * NOUT + c] = float(hQ[i * NOUT + c] * sc[i]);
  if (hipMemcpy(s->A, hA.data(), sizeof(float) * NFEAT * NOUT, hipMemcpyHostToDevice) != hipSuccess)
    return sfail(s, GW_EHIP, "skip upload");
  hipLaunchKernelGGL(k_residual, dim3(nblk(n * NOUT)), dim3(256), 0, st, feat, C, s->A, n, s->zmean, s->zstd, Z, 0);
  hipLaunchKernelGGL(k_colstats, dim3(NOUT), dim3(256), 0, st, Z, n, NOUT, s->zmean, s->zstd);
  hipLaunchKernelGGL(k_residual, dim3(nblk(n * NOUT)), dim3(256), 0, st, feat, C, s->A, n, s->zmean, s->zstd, Z, 1);
  if (hipStreamSynchronize(st) != hipSuccess) return sfail(s, GW_EHIP, "fit_skip");
  return GW_OK;
}

gw_status gw_surrogate_standardise(gw_surrogate* s, const double* feat, const float* C, int64_t n, float* Z, hipStream_t st) {
  if (!s || !feat || !C || !Z || n < 0) return GW_EINVAL;
  if (n == 0) return GW_OK;
  hipLaunchKernelGGL(k_residual, dim3(nblk(n * NOUT)), dim3(256), 0, st, feat, C, s->A, n, s->zmean, s->zstd, Z, 0);
  hipLaunchKernelGGL(k_residual, dim3(nblk(n * NOUT)), dim3(256), 0, st, feat, C, s->A, n, s->zmean, s->zstd, Z, 1);
  return slaunch(s, "standardise");
}

gw_status gw_surrogate_forward(gw_surrogate* s, const float* theta, int64_t B, float* out, hipStream_t st) {
  if (!s || !theta || !out || B < 1 || B > s->bmax) return GW_EINVAL;
  return mlp_infer(s, mlp_args(s, theta, B), out, nullptr, st);
}

// Gradients of the mean-squared loss for (theta, z) without an update.
// grads: device float [gw_surrogate_n_weights()] in the flat weight layout.
gw_status gw_surrogate_gradients(gw_surrogate* s, const float* theta, const float* z, int64_t B, float* grads, float* loss,
                                 hipStream_t st) {
  if (!s || !theta || !z || !grads || B < 1 || B > s->bmax) return GW_EINVAL;
  return mlp_train(s, theta, z, B, grads, loss, ParamArgs{}, st);
}

gw_status gw_surrogate_set_adam(gw_surrogate* s, double beta1, double beta2, double eps) {
  if (!s) return GW_EINVAL;
  if (!(beta1 >= 0.0 && beta1 < 1.0) || !(beta2 >= 0.0 && beta2 < 1.0) || !(eps > 0.0) || !std::isfinite(eps))
    return sfail(s, GW_EINVAL, "need 0 <= beta1, beta2 < 1 and eps > 0");
  s->beta1 = beta1;
  s->beta2 = beta2;
  s->eps = eps;
  return GW_OK;
}

gw_status gw_surrogate_train_step(gw_surrogate* s, const float* theta, const float* z, int64_t B, float lr,
                                  float weight_decay, float* loss, hipStream_t st) {
  if (!s || !theta || !z || B < 1 || B > s->bmax || !(lr >= 0.f) || !(weight_decay >= 0.f)) return GW_EINVAL;
  s->step += 1;
  // bias corrections 1/(1 - beta^t) in binary64 on the host
  ParamArgs u{};
  u.lr = lr;
  u.b1 = float(s->beta1);
  u.b2 = float(s->beta2);
  u.eps = float(s->eps);
  u.wd = weight_decay;
  u.c1 = float(1.0 / (1.0 - std::pow(s->beta1, double(s->step))));
  u.c2 = float(1.0 / (1.0 - std::pow(s->beta2, double(s->step))));
  return mlp_train(s, theta, z, B, nullptr, loss, u, st);
}

gw_status gw_surrogate_hidden(gw_surrogate* s, const float* theta, int64_t B, float* h3, hipStream_t st) {
  if (!s || !theta || !h3 || B < 1 || B > s->bmax) return GW_EINVAL;
  gw_status r = mlp_infer(s, mlp_args(s, theta, B), nullptr, s->hlast, st);
  if (r != GW_OK) return r;
  hipLaunchKernelGGL(k_bf16_to_f32, dim3(nblk(B * HID)), dim3(256), 0, st, s->hlast, B * HID, h3);
  return slaunch(s, "hidden");
}

gw_status gw_surrogate_set_head(gw_surrogate* s, const float* host_head, int64_t n) {
  if (!s || !host_head || n != HID + 1) return GW_EINVAL;
  if (hipMemcpy(s->head, host_head, sizeof(float) * (HID + 1), hipMemcpyHostToDevice) != hipSuccess) return GW_EHIP;
  return GW_OK;
}

// Ridge least squares of y = log10(max(mm, 1e-12)) (mm: measured mismatches,
// host, [n]) on the hidden features h3 (device, [n][HID]) plus a constant,
// with the penalty ridge * n on every coefficient; writes the head
// (synchronous).
gw_status gw_surrogate_fit_head(gw_surrogate* s, const float* h3_dev, const double* mm_host, int64_t n,
                                double ridge) {
  if (!s || !h3_dev || !mm_host || n < 1) return GW_EINVAL;
  if (!(ridge >= 0.0) || !std::isfinite(ridge)) return sfail(s, GW_EINVAL, "ridge must be finite and >= 0");
  std::vector<double> y_host(static_cast<size_t>(n));
  for (int64_t i = 0; i < n; ++i) {
    const double m = mm_host[i];
    if (!std::isfinite(m)) return sfail(s, GW_EINVAL, "non-finite mismatch");
    y_host[i] = std::log10(m > 1e-12 ? m : 1e-12);  // rounding can leave mm slightly below 0
  }
  std::vector<float> h(size_t(n) * HID);
  if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(h.data(), h3_dev, sizeof(float) * n * HID, hipMemcpyDeviceToHost) != hipSuccess)
    return sfail(s, GW_EHIP, "fit_head copy");
  const int D = HID + 1;
  std::vector<double> P(size_t(D) * D, 0.0), q(D, 0.0);
  for (int64_t i = 0; i < n; ++i) {
    double x[HID + 1];
    for (int j = 0; j < HID; ++j) x[j] = h[size_t(i) * HID + j];
    x[HID] = 1.0;
    for (int a = 0; a < D; ++a) {
      q[a] += x[a] * y_host[size_t(i)];
      for (int b2 = 0; b2 <= a; ++b2) P[size_t(a) * D + b2] += x[a] * x[b2];
    }
  }
  for (int a = 0; a < D; ++a)
    for (int b2 = a + 1; b2 < D; ++b2) P[size_t(a) * D + b2] = P[size_t(b2) * D + a];
  for (int a = 0; a < D; ++a) P[size_t(a) * D + a] += ridge * double(n);
  if (!chol_solve(P, D, q, 1)) return sfail(s, GW_EINVAL, "head: singular system");
  std::vector<float> hh(D);
  for (int a = 0; a < D; ++a) hh[a] = float(q[a]);
  return gw_surrogate_set_head(s, hh.data(), D);
}

// Node values [B][2][NN] (and predicted log10 mismatch [B]) for parameters.
gw_status gw_surrogate_nodes(gw_surrogate* s, const double* params, int64_t B, float* nodes, float* logmm, hipStream_t st) {
  if (!s || !params || !nodes || B < 0) return GW_EINVAL;
  if (B == 0) return GW_OK;
  for (int64_t b0 = 0; b0 < B; b0 += s->bmax) {
    const int64_t nb = std::min(s->bmax, B - b0);
    MlpArgs a = mlp_args(s, nullptr, nb);
    a.params = params;
    a.pB = B;
    a.b0 = b0;
    gw_status r = mlp_infer(s, a, s->zout, s->hlast, st);
    if (r != GW_OK) return r;
    ReconArgs ra{params, B, b0, s->zout, s->A, s->zmean, s->zstd, s->basis, s->mean, s->hlast, s->head,
                 nb, nodes + b0 * 2 * NN, logmm ? logmm + b0 : nullptr};
    hipLaunchKernelGGL(k_coefficients, dim3(unsigned(nb)), dim3(256), 0, st, ra, s->coef);
    hipLaunchKernelGGL(k_reconstruct, dim3(NN / 256, unsigned((nb + 31) / 32), 2), dim3(256), 0, st, ra,
                       static_cast<const float*>(s->coef));
  }
  return slaunch(s, "nodes");
}

gw_status gw_surrogate_waveform(gw_surrogate* s, const double* params, const float* nodes, int64_t B, float* hp, float* hc,
                                hipStream_t st) {
  if (!s || !params || !nodes || !hp || !hc || B < 0 || B > 0x7fffffff) return GW_EINVAL;
  if (B == 0) return GW_OK;
  SurrWaveArgs a{s->ctx->dc, params, B, nodes, s->ctx->k53, s->ctx->lnk3, hp, hc};
  const dim3 grid = dim3(unsigned(B));
  hipLaunchKernelGGL(k_surrogate_waveform, grid, dim3(256), 0, st, a);
  return slaunch(s, "k_surrogate_waveform");
}

gw_status gw_mismatch_max(gw_ctx* c, const float* ha, const float* hb, const float* psd, const double* params,
                          int64_t B, double* mm, hipStream_t st) {
  if (!c || B < 0) return GW_EINVAL;
  if (c->dc.precision == 2 || c->dc.N > 32768)
    return gw::ctx_fail(c, GW_EUNSUPPORTED, "gw_mismatch_max needs binary32 transforms and N <= 32768");
  if (B == 0) return GW_OK;  // the buffers of an empty batch may be NULL
  if (!ha || !hb || !psd || !mm) return gw::ctx_fail(c, GW_EINVAL, "NULL buffer");
  if (B > 0x7fffffff) return gw::ctx_fail(c, GW_EINVAL, "bad B");
  MismatchMaxArgs a{ha, hb, psd, B, c->dc.F, c->dc.kmin, c->dc.invT, params,
                    static_cast<const cpx<float>*>(c->tw_win), mm};
  const dim3 grid = dim3(unsigned(B));
  switch (c->dc.N / 2) {
    case 1024: hipLaunchKernelGGL((k_mismatch_max<1024>), grid, dim3(64), 0, st, a); break;
    case 2048: hipLaunchKernelGGL((k_mismatch_max<2048>), grid, dim3(128), 0, st, a); break;
    case 4096: hipLaunchKernelGGL((k_mismatch_max<4096>), grid, dim3(256), 0, st, a); break;
    case 8192: hipLaunchKernelGGL((k_mismatch_max<8192>), grid, dim3(512), 0, st, a); break;
    default: hipLaunchKernelGGL((k_mismatch_max<16384>), grid, dim3(1024), 0, st, a); break;
  }
  return gw::ctx_check_launch(c, "k_mismatch_max");
}

gw_status gw_mismatch(gw_ctx* c, const float* ha, const float* hb, const float* psd, const double* params, int64_t B,
                      double* mm, hipStream_t st) {
  if (!c || B < 0) return GW_EINVAL;
  if (B == 0) return GW_OK;  // the buffers of an empty batch may be NULL
  if (!ha || !hb || !psd || !mm) return gw::ctx_fail(c, GW_EINVAL, "NULL buffer");
  if (B > 0x7fffffff) return gw::ctx_fail(c, GW_EINVAL, "bad B");
  MismatchArgs a{ha, hb, psd, B, c->dc.F, c->dc.kmin, c->dc.invT, params, mm};
  hipLaunchKernelGGL(k_mismatch, dim3(unsigned(B)), dim3(256), 0, st, a);
  return gw::ctx_check_launch(c, "k_mismatch");
}

// Checkpoint file (host): magic "GWSURR2", then the basis, mean, skip path,
// standardisation and head, each layer's weights and biases, then the
// optimiser state: each layer's first and second moments of the weights and
// biases, the step counter (int64) and beta1, beta2, eps (binary64).  Files
// written before the optimiser state was kept ("GWSURR1") load with the
// moments and step counter reset.
static const char kMagic1[8] = {'G', 'W', 'S', 'U', 'R', 'R', '1', 0};
static const char kMagic2[8] = {'G', 'W', 'S', 'U', 'R', 'R', '2', 0};

gw_status gw_surrogate_save(gw_surrogate* s, const char* path) {
  if (!s || !path) return GW_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return sfail(s, GW_EHIP, "save: synchronise");
  FILE* f = std::fopen(path, "wb");
  if (!f) return sfail(s, GW_EINVAL, "cannot open file");
  auto put = [&](const void* dev, size_t bytes) {
    std::vector<char> h(bytes);
    if (hipMemcpy(h.data(), dev, bytes, hipMemcpyDeviceToHost) != hipSuccess) return false;
    return std::fwrite(h.data(), 1, bytes, f) == bytes;
  };
  auto put_host = [&](const void* p, size_t bytes) { return std::fwrite(p, 1, bytes, f) == bytes; };
  bool ok = put_host(kMagic2, 8) && put(s->basis, sizeof(float) * 2 * NBAS * NN) &&
            put(s->mean, sizeof(double) * 2 * NN) && put(s->A, sizeof(float) * NFEAT * NOUT) &&
            put(s->zmean, sizeof(float) * NOUT) && put(s->zstd, sizeof(float) * NOUT) && put(s->head, sizeof(float) * (HID + 1));
  for (int l = 0; l < NLAYER && ok; ++l)
    ok = put(s->W[l], sizeof(float) * layer_wn(l)) && put(s->b[l], sizeof(float) * layer_out(l));
  for (int l = 0; l < NLAYER && ok; ++l)
    ok = put(s->mW[l], sizeof(float) * layer_wn(l)) && put(s->vW[l], sizeof(float) * layer_wn(l)) &&
         put(s->mb[l], sizeof(float) * layer_out(l)) && put(s->vb[l], sizeof(float) * layer_out(l));
  const double hyper[3] = {s->beta1, s->beta2, s->eps};
  ok = ok && put_host(&s->step, sizeof(int64_t)) && put_host(hyper, sizeof(hyper));
  ok = (std::fclose(f) == 0) && ok;
  return ok ? GW_OK : sfail(s, GW_EHIP, "save failed");
}

gw_status gw_surrogate_load(gw_surrogate* s, const char* path) {
  if (!s || !path) return GW_EINVAL;
  FILE* f = std::fopen(path, "rb");
  if (!f) return sfail(s, GW_EINVAL, "cannot open file");
  auto get = [&](void* dev, size_t bytes) {
    std::vector<char> h(bytes);
    if (std::fread(h.data(), 1, bytes, f) != bytes) return false;
    return hipMemcpy(dev, h.data(), bytes, hipMemcpyHostToDevice) == hipSuccess;
  };
  char magic[8];
  bool ok = std::fread(magic, 1, 8, f) == 8;
  const bool v2 = ok && std::memcmp(magic, kMagic2, 8) == 0;
  ok = ok && (v2 || std::memcmp(magic, kMagic1, 7) == 0) &&
       get(s->basis, sizeof(float) * 2 * NBAS * NN) && get(s->mean, sizeof(double) * 2 * NN) &&
       get(s->A, sizeof(float) * NFEAT * NOUT) && get(s->zmean, sizeof(float) * NOUT) &&
       get(s->zstd, sizeof(float) * NOUT) && get(s->head, sizeof(float) * (HID + 1));
  for (int l = 0; l < NLAYER && ok; ++l) {
    ok = get(s->W[l], sizeof(float) * layer_wn(l)) && get(s->b[l], sizeof(float) * layer_out(l));
    if (ok)
      hipLaunchKernelGGL(k_weights_bf16, dim3(nblk(layer_wn(l))), dim3(256), 0, 0, s->W[l], layer_in(l), layer_out(l),
                         s->wf[l], s->wb[l]);
  }
  int64_t step = 0;
  double hyper[3] = {0.9, 0.999, 1e-8};
  if (v2) {
    for (int l = 0; l < NLAYER && ok; ++l)
      ok = get(s->mW[l], sizeof(float) * layer_wn(l)) && get(s->vW[l], sizeof(float) * layer_wn(l)) &&
           get(s->mb[l], sizeof(float) * layer_out(l)) && get(s->vb[l], sizeof(float) * layer_out(l));
    ok = ok && std::fread(&step, sizeof(int64_t), 1, f) == 1 && std::fread(hyper, sizeof(double), 3, f) == 3 &&
         step >= 0 && hyper[0] >= 0.0 && hyper[0] < 1.0 && hyper[1] >= 0.0 && hyper[1] < 1.0 && hyper[2] > 0.0;
  } else {
    for (int l = 0; l < NLAYER && ok; ++l)
      ok = hipMemset(s->mW[l], 0, sizeof(float) * layer_wn(l)) == hipSuccess &&
           hipMemset(s->vW[l], 0, sizeof(float) * layer_wn(l)) == hipSuccess &&
           hipMemset(s->mb[l], 0, sizeof(float) * layer_out(l)) == hipSuccess &&
           hipMemset(s->vb[l], 0, sizeof(float) * layer_out(l)) == hipSuccess;
  }
  std::fclose(f);
  if (!ok) return sfail(s, GW_EINVAL, "load failed (bad or truncated file)");
  s->step = step;
  s->beta1 = hyper[0];
  s->beta2 = hyper[1];
  s->eps = hyper[2];
  return hipDeviceSynchronize() == hipSuccess ? GW_OK : sfail(s, GW_EHIP, "load: synchronise");
}

}  // extern "C"

extern "C" gw_status gw_surrogate_set_state(gw_surrogate* s, const float* basis, const double* mean, const float* A,
                                            const float* zmean, const float* zstd, const float* head) {
  if (!s || !basis || !mean || !A || !zmean || !zstd || !head) return GW_EINVAL;
  bool ok = hipMemcpy(s->basis, basis, sizeof(float) * 2 * NBAS * NN, hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(s->mean, mean, sizeof(double) * 2 * NN, hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(s->A, A, sizeof(float) * NFEAT * NOUT, hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(s->zmean, zmean, sizeof(float) * NOUT, hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(s->zstd, zstd, sizeof(float) * NOUT, hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(s->head, head, sizeof(float) * (HID + 1), hipMemcpyHostToDevice) == hipSuccess;
  return ok ? GW_OK : sfail(s, GW_EHIP, "set_state");
}

extern "C" gw_status gw_surrogate_get_state(gw_surrogate* s, float* basis, double* mean, float* A, float* zmean,
                                            float* zstd, float* head) {
  if (!s || !basis || !mean || !A || !zmean || !zstd || !head) return GW_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return sfail(s, GW_EHIP, "get_state: synchronise");
  bool ok = hipMemcpy(basis, s->basis, sizeof(float) * 2 * NBAS * NN, hipMemcpyDeviceToHost) == hipSuccess &&
            hipMemcpy(mean, s->mean, sizeof(double) * 2 * NN, hipMemcpyDeviceToHost) == hipSuccess &&
            hipMemcpy(A, s->A, sizeof(float) * NFEAT * NOUT, hipMemcpyDeviceToHost) == hipSuccess &&
            hipMemcpy(zmean, s->zmean, sizeof(float) * NOUT, hipMemcpyDeviceToHost) == hipSuccess &&
            hipMemcpy(zstd, s->zstd, sizeof(float) * NOUT, hipMemcpyDeviceToHost) == hipSuccess &&
            hipMemcpy(head, s->head, sizeof(float) * (HID + 1), hipMemcpyDeviceToHost) == hipSuccess;
  return ok ? GW_OK : sfail(s, GW_EHIP, "get_state");
}
