// Per-item device code shared by the batch kernels and the persistent
// ragged kernels: the window item (rfft -> signal -> whiten -> irfft) and the
// Welch item, each run by the NC/16 threads of a (sub-)block on its own LDS
// planes.
#pragma once
#include <hip/hip_runtime.h>

#include "gw_fft.hpp"
#include "gw_physics.hpp"
#include "../../include/gwgen.h"

namespace gw {

// ---------------------------------------- window kernels (FFT of length N)
// Background offset of global sample index g in [0, span) (with ext_k sky
// positions per intrinsic draw, see draw_sample).
__device__ __forceinline__ int64_t draw_offset(uint64_t seed, uint64_t g, uint32_t ext_k, int64_t span) {
  const uint64_t gi = ext_k == 1u ? g : g / ext_k;
  return int64_t(floor(philox_uniform(seed, gi, 12u, uint32_t(g - gi * ext_k)) * double(span)));
}

// Where a batch's draws go.
struct DrawOut {
  double* params;      // [12][B]
  int64_t* offset;     // [B]
  float* params_f32;   // [12][B] or NULL
  WfScalars* wf;       // [B] waveform constants for the fused kernel, or NULL
  DetScalars* dsc;     // [B][D] antenna patterns and delays (with wf)
  uint32_t* status;    // [B] or NULL (set with wf only)
};

// Prior draws for global sample index g (the densities of Table 1 with the
// ranges in c), the window's background offset in [0, span), status
// initialisation, and the per-sample constants of the fused window kernel, by
// the kSetupLanes lanes of one group: lane r draws and transforms row r.
// Row 11 of the parameters receives p11.  With ext_k sky positions per
// intrinsic draw, g is sky position g % ext_k of intrinsic draw g / ext_k:
// every row is drawn at counter index g / ext_k, and alpha, delta, psi and
// the offset use the sub-counter g % ext_k (ext_k = 1: ordinary draws).
__device__ __forceinline__ double draw_row(const DevCfg& c, int r, double u) {
#pragma clang fp contract(off)
  if (r == 5) return acos(2.0 * u - 1.0);
  if (r == 7) return asin(2.0 * u - 1.0);
  if (c.approximant == 2) {
    // sine-Gaussian: f0 and Q uniform, hrss log-uniform
    if (r == 2) return exp(log(c.hrssr[0]) + u * (log(c.hrssr[1]) - log(c.hrssr[0])));
    if (r == 3 || r == 4) return 0.0;
  } else if (r == 4) {
    const double a3 = c.dl[0] * c.dl[0] * c.dl[0], b3 = c.dl[1] * c.dl[1] * c.dl[1];
    return cbrt(a3 + u * (b3 - a3));
  }
  const bool burst = c.approximant == 2;
  const double lo = r == 0 ? (burst ? c.f0r[0] : c.mc[0]) : r == 1 ? (burst ? c.Qr[0] : c.q[0]) : c.chi[0];
  const double hi = r == 0 ? (burst ? c.f0r[1] : c.mc[1]) : r == 1 ? (burst ? c.Qr[1] : c.q[1]) : c.chi[1];
  if (r <= 3) return lo + u * (hi - lo);
  if (r == 8) return kPi * u;
  if (r == 10) return c.T - 1.5 + u * 1.0;
  return 2.0 * kPi * u;
}

__device__ __forceinline__ void draw_sample(const DevCfg& c, uint64_t seed, uint64_t g, int64_t i, int64_t B,
                                            int64_t span, double p11, const DrawOut& o, int lane, uint32_t ext_k = 1u) {
  const uint64_t gi = ext_k == 1u ? g : g / ext_k;
  const uint32_t j = uint32_t(g - gi * ext_k);
  const double mine =
      lane < 11 ? draw_row(c, lane, philox_uniform(seed, gi, uint32_t(lane), (lane >= 6 && lane <= 8) ? j : 0u)) : p11;
  if (lane < 12) {
    o.params[lane * B + i] = mine;
    if (o.params_f32) o.params_f32[lane * B + i] = float(mine);
  } else if (lane == 12) {
    o.offset[i] = draw_offset(seed, g, ext_k, span);
  }
  if (!o.wf) return;
  double p[11];
#pragma unroll
  for (int r = 0; r < 11; ++r) p[r] = lane_value(mine, r);
  WfScalars w = {};
  WfModel model;  // (of no use here)
  SkyAngles sky;
  wf_setup(p, c, lane, w, model, sky);
  if (lane == 0) {
    o.wf[i] = w;
    if (o.status) {
      // sine-Gaussian: f0 + 5/(pi tau) beyond Nyquist
      const bool cut = c.approximant == 2 ? p[0] + 5.0 / (kPi * (p[1] / (sqrt(2.0) * kPi * p[0]))) > 0.5 * c.fs
                                          : w.cut_nyquist != 0;
      o.status[i] = cut ? GW_STATUS_CUT_AT_NYQUIST : 0u;
    }
  }
  if (lane < c.n_det) o.dsc[i * c.n_det + lane] = det_response(c.det[lane], sky, w.tc);
}

// Load through the constant address space: for memory that no thread writes
// while the kernel runs.  A uniform address then becomes a scalar load even
// after earlier stores in the same kernel.
template <class T>
__device__ __forceinline__ T load_const(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole 32-bit words");
  typedef const __attribute__((address_space(4))) uint32_t* cword_ptr;
  const cword_ptr q = (cword_ptr)(p);
  T v;
  uint32_t* o = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
  for (int i = 0; i < int(sizeof(T) / 4); ++i) o[i] = q[i];
  return v;
}

struct WinArgs {
  DevCfg cf;
  const float* src;       // strain [B][D][N] (SRC 0, 2) or background (SRC 1)
  int64_t L_bg;
  const float* bg;        // background for inject (SRC 2)
  const int64_t* offset;
  const double* params;
  int64_t B;
  const float* psd;       // [B][D][Fw]
  float* out;
  uint32_t* status;
  const double* kcbrt;
  const double* lnk3;
  const double* k53;      // k^(-5/3)
  const void* tw;         // pass twiddle tables of the N/2-point transform
  const void* twr;        // cpx<T>[N/4 + 1], exp(-2 pi i k / N)
  const WfScalars* wf;    // [B] (SRC 1, 3)
  const DetScalars* dsc;  // [B][D] (SRC 1, 3)
  const float* nodes;     // [B][2][1024] surrogate node values (SRC 3)
  const float* logmm;     // [B] predicted log10 mismatch (SRC 3)
  float logmm_max;        // fallback threshold (SRC 3)
  int crop;               // samples dropped at each end of the output (SRC 4; even)
  float* out2;            // SRC 5: the reference views [B][D][N]
  double t_ref;           // SRC 5: the reference view's signal time
};

// Surrogate node grid: 1024 points log-spaced in Mf over [2e-3, 0.2].
constexpr int kSurrNodes = 1024;
constexpr double kSurrLnMfLo = -6.2146080984221914;   // ln(2e-3)
constexpr double kSurrDlog = 4.6051701859880914 / 1023.0;  // ln(0.2/2e-3)/(NN-1)

// Lower PSD bin for window bin k, clamped so that it and the next bin exist
// for every k in [0, N/2] (the PSD has L/2 + 1 bins, L/2 = (N/2) / ratio).
__device__ __forceinline__ int psd_index(const DevCfg& cf, int k, int NC) {
  return min(k >> cf.log2_ratio, (NC >> cf.log2_ratio) - 1);
}

// The PSD values around window bins k and NC - k.
struct PsdAround { float lo[2], hi[2]; };
__device__ __forceinline__ PsdAround psd_around(const DevCfg& cf, const float* psd, int k, int NC) {
  PsdAround q;
  __builtin_memcpy(q.lo, psd + psd_index(cf, k, NC), 8);
  __builtin_memcpy(q.hi, psd + psd_index(cf, NC - k, NC), 8);
  return q;
}

// S at window bin k from the values around it: t s1 + (1 - t) s0, two terms of
// one sign, so that where the PSD falls steeply the sum is as accurate as its
// terms (as s0 + t (s1 - s0), its error was up to N/L times larger).
template <class T> __device__ __forceinline__ T psd_at(const DevCfg& cf, const float* s, int k) {
  const T t = T(k & (cf.ratio - 1)) * T(cf.inv_ratio);
  return fma_t(t, T(s[1]), fma_t(-t, T(s[0]), T(s[0])));
}

// Whitening factor 1/sqrt(fs S/2) for a kept bin's PSD value S; sets status
// bits.  (The root is taken of fs S/2 and not of S: the hardware's reads a
// subnormal argument as zero.)
template <class T>
__device__ __forceinline__ T psd_gain(const DevCfg& cf, T S, bool kept, uint32_t& flag) {
  const bool good = S > T(0) && S < T(INFINITY);
  if (kept && !good) flag |= isfinite(S) ? GW_STATUS_NONPOSITIVE_PSD : GW_STATUS_NONFINITE_PSD;
  return kept && good ? rsqrt_t(T(cf.fs) * T(0.5) * S) : T(0);
}

// Whitening factors of bins k and NC - k, k in [0, NC/2].
template <class T>
__device__ __forceinline__ void psd_gains(const DevCfg& cf, const PsdAround& q, int k, int NC, uint32_t& flag, T* gk, T* gm) {
  const bool inner = k != 0;  // bins 0 and NC are dropped
  *gk = psd_gain<T>(cf, psd_at<T>(cf, q.lo, k), inner && k >= cf.kmin, flag);
  *gm = psd_gain<T>(cf, psd_at<T>(cf, q.hi, NC - k), inner && NC - k >= cf.kmin, flag);
}

// Whitening factor for window bin k in [0, N/2] (zero outside the kept band).
template <class T>
__device__ __forceinline__ T whiten_gain(const DevCfg& cf, const float* psd, int k, int NC, uint32_t& flag) {
  const T S = psd_at<T>(cf, psd + psd_index(cf, k, NC), k);
  return psd_gain<T>(cf, S, k > 0 && k < NC && k >= cf.kmin, flag);
}

// Gain g = filt[k] of a precomputed whitening filter; sets status bits.
template <class T>
__device__ __forceinline__ T filter_gain_at(float g, uint32_t& flag) {
  if (!isfinite(g)) { flag |= GW_STATUS_NONFINITE_PSD; return T(0); }
  return T(g);
}

// Real-spectrum unpack of the packed bins A = Z_k and B = Z_(NC-k), with
// W = exp(-2 pi i k / N): twice the real input's spectrum at k and NC - k.
template <class T>
__device__ __forceinline__ void unpack_pair(cpx<T> A, cpx<T> B, cpx<T> W, cpx<T>* Xk, cpx<T>* Xm) {
  const T sx = A.x + B.x, sy = A.y - B.y, dx = A.x - B.x, dy = A.y + B.y;  // A + conj B, A - conj B
  // X_k = s - i W d, X_m = conj(s + i W d)
  *Xk = {fma_t(W.x, dy, fma_t(W.y, dx, sx)), fma_t(-W.x, dx, fma_t(W.y, dy, sy))};
  *Xm = {fma_t(-W.x, dy, fma_t(-W.y, dx, sx)), fma_t(-W.x, dx, fma_t(W.y, dy, -sy))};
}

// The inverse packing: twice Z'_k and Z'_(NC-k) from the spectrum Y_k = gk Xk,
// Y_m = gm Xm at both bins.  (Products and sums are fused explicitly, so that
// every kernel that includes this rounds alike.)
template <class T>
__device__ __forceinline__ void repack_pair(cpx<T> Xk, T gk, cpx<T> Xm, T gm, cpx<T> W, cpx<T>* zk, cpx<T>* zm) {
  const T mx = gm * Xm.x, my = gm * Xm.y;
  const T px = fma_t(gk, Xk.x, mx), py = fma_t(gk, Xk.y, -my);  // p = Y_k + conj Y_m
  const T dx = fma_t(gk, Xk.x, -mx), dy = fma_t(gk, Xk.y, my);  // d = Y_k - conj Y_m
  // q = conj(W) d; Z'_k = p + i q, Z'_m = conj(p) + i conj(q)
  *zk = {fma_t(-W.x, dy, fma_t(W.y, dx, px)), fma_t(W.x, dx, fma_t(W.y, dy, py))};
  *zm = {fma_t(T(2), px, -zk->x), fma_t(T(-2), py, zk->y)};
}

// What unpack_pair and repack_pair leave out of a whitened window, applied where
// it is stored: 1/2 each for the two packings and the inverse transform's 1/NC.
template <class T> __device__ __forceinline__ T whitened_scale(int NC) { return T(0.25) / T(NC); }

// The detector's projection of one item: the signal is added to twice the
// spectrum, so the antenna factors carry 2 fs.
template <class T> struct Projection {
  T cpl, cxx;
  double tauT;  // time shift in windows
};

// Projected sine-Gaussian at bin k: sg_G0 [G(f - f0)(cpl - i cxx) e^{-2 pi i rm}
// + G(f + f0)(cpl + i cxx) e^{-2 pi i rp}], rm/rp = k tau/T -/+ phi0/(2 pi).
template <class T, class TP>
__device__ __forceinline__ cpx<T> burst_bin(const DevCfg& cf, const WfScalars& w, const Projection<T>& pr, int k) {
  const T cpl = pr.cpl, cxx = pr.cxx;
  const double f = double(k) * cf.invT;
  const T xm = T(f - w.sg_f0), xp = T(f + w.sg_f0);
  const T gm = exp(-T(w.sg_pt2) * xm * xm), gp = exp(-T(w.sg_pt2) * xp * xp);
  const TP base = frac_product(TP(k), TP(pr.tauT));
  T sm, cm, sp, cp;
  sincos_rev(T(frac1(base - TP(w.sg_rphi))), &sm, &cm);
  sincos_rev(T(frac1(base + TP(w.sg_rphi))), &sp, &cp);
  const T A = T(w.sg_G0);
  return {A * (gm * (cpl * cm - cxx * sm) + gp * (cpl * cp + cxx * sp)),
          A * (gp * (cxx * cp - cpl * sp) - gm * (cpl * sm + cxx * cm))};
}

// Adds the projected signal (plain model, generated in registers) at window
// bin k to X.  powers(k) gives the bin's powers.
template <class T, class TP, bool FULL, class Powers>
__device__ __forceinline__ void add_signal(const DevCfg& cf, const WfScalars& w, const Projection<T>& pr, int k,
                                           Powers powers, cpx<T>* X) {
  if (k <= 0 || k < cf.kmin || k >= w.kend) return;
  if (cf.approximant == 2) {
    *X = cadd(*X, burst_bin<T, TP>(cf, w, pr, k));
    return;
  }
  TP rev;
  T A;
  bin_polar<T, TP, FULL>(w, k, powers(k), &rev, &A);
  rev = frac1(fma_t(TP(k), TP(pr.tauT), rev));
  T s, c;
  sincos_rev(T(rev), &s, &c);
  // A (cpl - i cxx)(c - i s)
  s *= A;
  c *= A;
  *X = {fma_t(pr.cpl, c, fma_t(-pr.cxx, s, X->x)), fma_t(-pr.cpl, s, fma_t(-pr.cxx, c, X->y))};
}

// Node values staged in LDS: typed as such, so that their gathers compile to
// LDS reads rather than generic (flat) loads, which would also wait for the
// global loads issued ahead.
typedef const __attribute__((address_space(3))) float* lds_cfptr;

// The same from surrogate node values: binary64 Newtonian phase + interpolated
// phase residual (revolutions), amplitude A_N(f_k) times the interpolated ratio.
template <class T>
__device__ __forceinline__ void add_signal_surr(const DevCfg& cf, const WinArgs& a, const WfScalars& w, lds_cfptr nd,
                                                const Projection<T>& pr, int k, cpx<T>* X) {
  if (k <= 0 || k < cf.kmin || k >= w.kend) return;
  const double lk3 = a.lnk3[k], k53 = a.k53[k];
  // u = (ln(Ms k / T) - ln Mf_lo) / dlog, ln(Ms/T) = 3 ln v1 - ln pi
  const float u = float((3.0 * w.lnv1 - 1.1447298858494002 - kSurrLnMfLo + 3.0 * lk3) * (1.0 / kSurrDlog));
  const float uc = fminf(fmaxf(u, 0.f), float(kSurrNodes - 1));
  const int i = min(int(uc), kSurrNodes - 2);
  const float tt = uc - float(i);
  const float ratio = (1.f - tt) * nd[i] + tt * nd[i + 1];
  const float dpsi = (1.f - tt) * nd[kSurrNodes + i] + tt * nd[kSurrNodes + i + 1];
  // Newtonian phase cN k^(-5/3) from the table: one binary64 product per bin
  double rev = w.cN * k53 + double(dpsi) * (1.0 / (2.0 * kPi)) + w.pconst + double(k) * pr.tauT;
  rev = frac1(rev);
  T s, c;
  sincos_rev(T(rev), &s, &c);
  // A_N(f_k) = A0T k^(-7/6) = A0T k^(-5/3) k^(1/2)
  const T kf = T(k);
  const T A = T(w.A0T) * T(k53) * (kf * rsqrt_t(kf)) * T(ratio);
  s *= A;
  c *= A;
  *X = {fma_t(pr.cpl, c, fma_t(-pr.cxx, s, X->x)), fma_t(-pr.cpl, s, fma_t(-pr.cxx, c, X->y))};
}

// One window item (sample b, detector d) handled by the NC/16 threads t of a
// (sub-)block, with its own LDS planes.
// SRC 0: whiten strain (x = strain row).  SRC 1: background + in-register
// signal + whiten (x = background at o + P).  SRC 3: as SRC 1 with the signal
// from surrogate node values (plain model where the predicted mismatch
// exceeds the threshold).  SRC 2: inject (hrow = hdet row, nz = noise window).
// SRC 4: as SRC 1 whitened with a fixed per-run filter (psd = filter row of
// N/2 + 1 gains), storing samples [crop, N - crop) only.  SRC 5: the view
// pair of one item: as SRC 1 into o, then, from the same noise spectrum kept
// in registers, the same window with the signal at t_ref into o2.
// `active` false: compute on the given (valid) item but store nothing, so
// that idle sub-blocks still meet every block barrier.
// Bins t + NT j, j < 8, stay in registers from the forward transform to the
// inverse one and only the upper half of the spectrum, their partners, goes
// through LDS, as far as registers allow (SRC 5 has none left): a quarter of
// the exchanges between the transforms were of bins a thread gave itself.
// 2048 samples with a run filter 278.9 -> 275.7 us (280 since the transforms'
// first stages take sines, see kSineTable).
// Bound by its vector arithmetic, most of it in the pairs' loop: of 820
// instructions for two pairs, 120 went with the phase and the amplitude from
// one table of k^(-5/3), products summed as fused steps, the factors common
// to all bins moved to the store and each PSD neighbour read once as eight
// bytes.  2048 samples of 3 detectors, N = 16384: 361 us before, 344 then (SRC
// 1; 347 since the gain's root takes fs S/2 and the first stages take sines);
// view pairs of 301 samples 112 and 105; 32 samples, N = 524288, on the path for
// long windows (the pairs of k_long_rowpair) 255 and 248.
template <class T, class TP, bool FULL, int NC, int SRC, int ORD>
__device__ __forceinline__ void window_item(const DevCfg& cf, const WinArgs& a, int t, int64_t b, int d,
                                            const float* x, const float* hrow, const float* nz, const float* psd,
                                            float* o, const cpx<T>* twtab, const cpx<T>* twr, T* sre, T* sim,
                                            bool active, uint32_t* sflag, float* snodes = nullptr,
                                            float* o2 = nullptr) {
  constexpr int NT = NC / 16;
  static_assert(SRC >= 0 && SRC <= 5, "source");
  constexpr bool SIG = SRC == 1 || SRC == 5;  // in-register plain-model signal
  PassTwiddle<T, NC, ORD> tw{twtab};
  if constexpr (SRC == 3) {
    // the sample's node values go to LDS once (snodes: 2 x 1024 floats of
    // LDS); the barriers of the forward transform below make them visible to
    // the whole (sub-)block
    const float* src = a.nodes + b * 2 * kSurrNodes;
    for (int i = t; i < 2 * kSurrNodes; i += NT) snodes[i] = src[i];
  }
  constexpr bool kOwn = SRC != 5;  // SRC 5 keeps the noise spectrum in registers instead
  constexpr int RL = PlanEnds<NC, ORD>::RLAST;
  cpx<T> own[kOwn ? 8 : 1];
  cpx<T> v[16];
  uint32_t flag = 0;
  if constexpr (SRC != 2) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      float2 q;
      __builtin_memcpy(&q, x + 2 * (t + NT * j), sizeof(q));
      v[fft_in_slot<NC, ORD>(j)] = {T(q.x), T(q.y)};
    }
    // fresh lane indices and a fresh table pointer per transform: otherwise
    // the compiler shares the forward and inverse transforms' index
    // arithmetic and twiddle loads and keeps them live in between
    block_fft<T, NC, -1, false, ORD>(v, sre, sim, fresh_lane(t), tw);
    lds_barrier();
    const int tn = fresh_lane(t);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int j = e / RL + (e % RL) * (16 / RL);  // v[e] is bin t + NT j
      if (kOwn && j < 8) {
        own[j] = v[e];
        if (j == 0 && t == 0) {  // bin 0 pairs with itself
          sre[0] = v[e].x;
          sim[0] = v[e].y;
        }
        continue;
      }
      const int i = lpad<T>(fft_out_index<NC, ORD>(tn, e));
      sre[i] = v[e].x;
      sim[i] = v[e].y;
    }
    lds_barrier();
  }
  // SRC 5: this thread's share of the noise spectrum, for the second view
  cpx<T> keep[SRC == 5 ? 16 : 1];
  if constexpr (SRC == 5) {
#pragma unroll
    for (int e = 0; e < 16; ++e) keep[e] = v[e];
  }

  Projection<T> pr = {T(0), T(0), 0.0};
  WfScalars wsh;
  if constexpr (SIG || SRC == 3 || SRC == 4) wsh = load_const(a.wf + b);
  bool use_surr = false;
  lds_cfptr nd = nullptr;
  if constexpr (SRC == 3) {
    // a NaN prediction fails the test and falls back to the plain model
    use_surr = load_const(a.logmm + b) <= a.logmm_max;
    nd = (lds_cfptr)snodes;  // staged before the forward transform
    if (active && !use_surr && t == 0 && d == 0 && a.status)
      atomicOr(a.status + b, uint32_t(GW_STATUS_SURROGATE_FALLBACK));
  }
  double tauT_ref = 0.0;  // SRC 5: the reference view's time shift
  if constexpr (SIG || SRC == 3 || SRC == 4) {
    const DetScalars dsh = load_const(a.dsc + (b * cf.n_det + d));
    pr = {T(cf.fs * dsh.fp * (1.0 + wsh.cosi * wsh.cosi)), T(2.0 * cf.fs * dsh.fx * wsh.cosi), dsh.tau * cf.invT};
    if constexpr (SRC == 5) tauT_ref = (dsh.tau - wsh.tc + a.t_ref) * cf.invT;  // same delays, signal at t_ref
  }
  auto powers = [&](int k) { return BinPowers{a.kcbrt[k], a.lnk3[k], a.k53[k]}; };
  const float2* hsrc = reinterpret_cast<const float2*>(hrow);

  // Global inputs of the pair (k, NC - k): the twiddle and what the two bins
  // need (PSD values, filter gains, or the signal to inject), fetched one
  // pair ahead so that their latency overlaps the previous pair's work.
  struct PairIn {
    cpx<T> W;
    float g[4];
  };
  auto fetch = [&](int k) {
    k = min(k, NC / 2);
    const int km = NC - k;
    PairIn q;
    q.W = twr[k];  // exp(-2 pi i k / N)
    if constexpr (SRC == 2) {
      const float2 h0 = hsrc[k], h1 = hsrc[km];
      q.g[0] = h0.x;
      q.g[1] = h0.y;
      q.g[2] = h1.x;
      q.g[3] = h1.y;
    } else if constexpr (SRC == 4) {
      q.g[0] = psd[k];
      q.g[1] = psd[km];
      q.g[2] = q.g[3] = 0.f;
    } else {
      const PsdAround p = psd_around(cf, psd, k, NC);
      q.g[0] = p.lo[0];
      q.g[1] = p.lo[1];
      q.g[2] = p.hi[0];
      q.g[3] = p.hi[1];
    }
    return q;
  };
  // the pair's spectrum values (k, NC - k)
  auto load_bin = [&](int k) {
    const int i = lpad<T>(k & (NC - 1));
    return cpx<T>{sre[i], sim[i]};
  };
  auto load_pair = [&](int k, int u, cpx<T>& A, cpx<T>& Bm) {
    if constexpr (SRC != 2) {
      if constexpr (kOwn) A = own[u];
      else A = load_bin(k);
      Bm = load_bin(NC - k);
    }
  };
  // unpack, signal, gain and repack of the pair: zk, zm go to bins k, NC - k
  // (both scaled, see whitened_scale)
  auto pair_out = [&](const PairIn& cur, int k, cpx<T> A, cpx<T> Bm, cpx<T>& zk, cpx<T>& zm) {
    const int km = NC - k;
    cpx<T> Yk, Ym;
    T gk = T(1), gm = T(1);
    if constexpr (SRC == 2) {
      Yk = {T(cur.g[0]), T(cur.g[1])};
      Ym = {T(cur.g[2]), T(cur.g[3])};
      if (k == 0) { Yk.y = T(0); Ym.y = T(0); }  // irfft ignores Im at DC and Nyquist
    } else {
      unpack_pair<T>(A, Bm, cur.W, &Yk, &Ym);
      bool plain = SIG || SRC == 4;
      if constexpr (SRC == 3) {
        plain = !use_surr;
        if (use_surr) {
          add_signal_surr<T>(cf, a, wsh, nd, pr, k, &Yk);
          add_signal_surr<T>(cf, a, wsh, nd, pr, km, &Ym);
        }
      }
      if (plain) {
        add_signal<T, TP, FULL>(cf, wsh, pr, k, powers, &Yk);
        add_signal<T, TP, FULL>(cf, wsh, pr, km, powers, &Ym);
      }
      if constexpr (SRC == 4) {
        // fixed per-run filter row [NC + 1] (zero outside the kept band)
        gk = filter_gain_at<T>(cur.g[0], flag);
        gm = filter_gain_at<T>(cur.g[1], flag);
      } else {
        psd_gains<T>(cf, PsdAround{{cur.g[0], cur.g[1]}, {cur.g[2], cur.g[3]}}, k, NC, flag, &gk, &gm);
      }
    }
    repack_pair<T>(Yk, gk, Ym, gm, cur.W, &zk, &zm);
  };
  auto store_bin = [&](int k, cpx<T> z) {
    const int i = lpad<T>(k);
    sre[i] = z.x;
    sim[i] = z.y;
  };
  auto store_pair = [&](int k, int u, cpx<T> zk, cpx<T> zm) {
    const int km = NC - k;
    if constexpr (kOwn) own[u] = zk;
    else store_bin(k, zk);
    if (k != 0 && km != k) store_bin(km, zm);
  };

  // pairs, inverse transform and store of one output window ov
  auto emit = [&](float* ov) {
  // pairs (k, NC - k) for k = t + NT i in [0, NC/2] (NC/2 = 8 NT): two per
  // loop trip, whose LDS reads are issued together and whose arithmetic
  // chains interleave; the last one (k = NC/2) belongs to thread 0 alone
  PairIn n0 = fetch(t), n1 = fetch(t + NT);
#pragma unroll 1
  for (int i = 0; i < 8; i += 2) {
    const int k0 = t + NT * i, k1 = k0 + NT;
    const PairIn c0 = n0, c1 = n1;
    n0 = fetch(k0 + 2 * NT);
    n1 = fetch(k1 + 2 * NT);
    cpx<T> A0 = {}, B0 = {}, A1 = {}, B1 = {}, z0k, z0m, z1k, z1m;
    load_pair(k0, 0, A0, B0);
    load_pair(k1, 1, A1, B1);
    pair_out(c0, k0, A0, B0, z0k, z0m);
    pair_out(c1, k1, A1, B1, z1k, z1m);
    store_pair(k0, 0, z0k, z0m);
    store_pair(k1, 1, z1k, z1m);
    if constexpr (kOwn) {  // the next two to the front
      const cpx<T> o0 = own[0], o1 = own[1];
#pragma unroll
      for (int j = 0; j < 6; ++j) own[j] = own[j + 2];
      own[6] = o0;
      own[7] = o1;
    }
  }
  if (t == 0) {  // n0 = fetch(NC/2)
    cpx<T> A = {}, zk, zm;
    if constexpr (SRC != 2) A = load_bin(NC / 2);
    pair_out(n0, NC / 2, A, A, zk, zm);
    store_bin(NC / 2, zk);
  }
  lds_barrier();
  if constexpr (kOwn) {
    const int tn = fresh_lane(t);
#pragma unroll
    for (int j = 0; j < 16; ++j) v[fft_in_slot<NC, ORD>(j)] = j < 8 ? own[j & 7] : load_bin(tn + NT * j);
    lds_barrier();
  }
  block_fft<T, NC, +1, !kOwn, ORD>(v, sre, sim, fresh_lane(t), PassTwiddle<T, NC, ORD>{opaque(twtab)});
  const T sc = SRC == 2 ? T(0.5) / T(NC) : whitened_scale<T>(NC);
  if (active) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int n = fft_out_index<NC, ORD>(t, e);
      float2 y = {float(v[e].x * sc), float(v[e].y * sc)};
      if constexpr (SRC == 2) {
        y.x += nz[2 * n];
        y.y += nz[2 * n + 1];
      }
      if constexpr (SRC == 4) {
        // cropped store: samples [crop, N - crop), crop even
        const int m = n - (a.crop >> 1);
        if (m >= 0 && m < NC - a.crop) reinterpret_cast<float2*>(ov)[m] = y;
      } else {
        reinterpret_cast<float2*>(ov)[n] = y;
      }
    }
  }
  };
  emit(o);
  if constexpr (SRC == 5) {
    // reference view: the noise spectrum back to LDS, the signal at t_ref
    lds_barrier();  // the inverse transform's last LDS reads are done
    const int tk = fresh_lane(t);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int i = lpad<T>(fft_out_index<NC, ORD>(tk, e));
      sre[i] = keep[e].x;
      sim[i] = keep[e].y;
    }
    lds_barrier();
    pr.tauT = tauT_ref;
    emit(o2);
  }
  if (active && flag) atomicOr(sflag, flag);
}

// a + b = s + e exactly (s the rounded sum)
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
  s = a + b;
  const double bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

// A binary64 sum h with the rounding errors of its additions, l.
struct PairSum { double h, l; };
__device__ __forceinline__ PairSum sum_add(PairSum a, PairSum b) {
  PairSum r;
  double e;
  two_sum(a.h, b.h, r.h, e);
  r.l = (a.l + b.l) + e;
  return r;
}
__device__ __forceinline__ double sum_add(double a, double b) { return a + b; }
__device__ __forceinline__ float sum_add(float a, float b) { return a + b; }
// times a power of two
__device__ __forceinline__ PairSum sum_scale(PairSum a, double c) { return {a.h * c, a.l * c}; }
__device__ __forceinline__ double sum_scale(double a, double c) { return a * c; }
__device__ __forceinline__ float sum_scale(float a, float c) { return a * c; }
__device__ __forceinline__ double sum_value(PairSum a) { return a.h + a.l; }
__device__ __forceinline__ double sum_value(double a) { return a; }
__device__ __forceinline__ float sum_value(float a) { return a; }

// Welch sums of (sample, detector) stretches x = background + o, by the NC/16
// threads t of a (sub-)block: periodic-Hann segments of L = NC samples at
// stride L/2.  Segments 2p and 2p+1 go through ONE complex FFT as real and
// imaginary parts; since |A_k|^2 + |B_k|^2 = (|X_k|^2 + |X_{L-k}|^2)/2 for
// X = FFT(a + i b), the accumulated |X|^2 is folded once at the end.
// With ACC wider than T (mixed precision) every transform's |X|^2 is added
// to ACC totals.  In binary32 throughout it is summed in two levels, runs of
// kRun transforms and then the run sums, so that the rounding error grows with
// kRun + K/(2 kRun) terms rather than K/2.  In binary64 throughout the
// additions' rounding errors are summed beside the totals (PairSum).  The fold
// and the normalisation are done in ACC.
//
// A stretch may be cut anywhere and its pieces' sums added (WelchCut) without
// a change in the result, because the sums are exact: binary32 terms in
// binary64 as long as none but zeros is below 2^-29 of the sum, binary64 terms
// in a PairSum down to 2^-49.  (A smaller term leaves a rounding at the sum's
// last place, which the result's own to binary32 shows in one of 10^8 such
// bins.  Plain binary64 sums of binary64 terms did so in every bin.  The
// errors' sum costs five more operations a bin; 300 stretches of 32 pairs of
// L = 4096 take 112 us with it, 101 without.)
//
// The kernel is bound by the issue of vector instructions: per pair and thread
// 32 for the window, 148 + 192 + 192 for the three radix-16 passes and 64 for
// the sums.  The matrix cores do not help: binary32 MFMA shares the vector
// units' multipliers, and a first pass as 32 products of 16 x 16 x 4 (575
// vector instructions left) took 1.20 against 0.93 ms at 6144 items of K = 63.
template <int NC> struct WelchTab {  // the table of one L = NC, in values of T
  static constexpr int hann = 2 * (PlanTw<NC, 0>::size + PlanTw<NC, 1>::size);  // pass tables, then sin^2(pi n / L)
  static constexpr int size = hann + NC / 2;                                    // for n < L/2
};

template <class T, class ACC, int NC, int ORD> struct WelchItem {
  static constexpr int NT = NC / 16, LS = LdsSize<NC>::value;
  static constexpr bool kWide = sizeof(ACC) > sizeof(T);
  static constexpr int kRun = 16;
  static constexpr bool kPair = sizeof(T) == 8;  // PairSum totals
  using Sum = std::conditional_t<kPair, PairSum, ACC>;
  static_assert(NC * sizeof(Sum) <= 2 * LS * sizeof(T), "fold buffer must fit in the FFT buffer");
  // sin^2 window at n = t + NT r, r < 8; half a segment later it is
  // cos^2 = 1 - sin^2, applied as x - w x
  T w[8];
  // binary64: with the twiddles held, a thread took 290 registers, one wave to
  // a SIMD; 300 stretches of 32 pairs of L = 4096 took 131 us, with two
  // waves 101 (before the sums carried their errors)
  static constexpr bool kLate = sizeof(T) == 8;
  std::conditional_t<kLate, LateTwiddle<T, NC, ORD>, HeldTwiddle<T, NC, ORD>> tw;
  ACC tot[16];
  T run[kWide ? 1 : 16];  // binary64: the totals' rounding errors
  int t;
  T *sre, *sim;

  __device__ __forceinline__ WelchItem(const T* tab, int t_, T* sre_, T* sim_) : t(t_), sre(sre_), sim(sim_) {
#pragma unroll
    for (int r = 0; r < 8; ++r) w[r] = tab[WelchTab<NC>::hann + t + NT * r];
    tw.init(reinterpret_cast<const cpx<T>*>(tab), t);
  }

  // |X|^2 of transform p
  __device__ __forceinline__ void add_power(const cpx<T>* v, int p) {
    if constexpr (kWide) {
#pragma unroll
      for (int e = 0; e < 16; ++e) tot[e] += ACC(fma_t(v[e].y, v[e].y, v[e].x * v[e].x));
    } else if constexpr (kPair) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        // (both addends are at least 0: the larger one's error is none)
        const double p2 = fma_t(v[e].y, v[e].y, v[e].x * v[e].x), s = tot[e] + p2;
        run[e] += __builtin_fmin(tot[e], p2) - (s - __builtin_fmax(tot[e], p2));
        tot[e] = s;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) run[e] = fma_t(v[e].y, v[e].y, fma_t(v[e].x, v[e].x, run[e]));
      if (p % kRun == kRun - 1) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          tot[e] += run[e];
          run[e] = T(0);
        }
      }
    }
  }

  __device__ __forceinline__ void load_half(const float* half, float* v) const {
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = half[t + NT * r];
  }

  // Sums of the segment pairs p0 <= p < p1 of the stretch x (K segments; with
  // K odd the last pair holds one).  Pair p covers [p L, p L + 3L/2): its first
  // half segment was read by pair p-1, and the next pair's two new ones are
  // requested before the current transform so that their latency hides behind
  // it (in the last trip, or for a single segment, half segments that were
  // read already are requested again, so that no branch splits the loop).
  __device__ __forceinline__ void pairs(const float* x, int K, int p0, int p1) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      tot[e] = ACC(0);
      if constexpr (!kWide) run[e] = T(0);
    }
    float cur[8], na[8], nb[8];
    // half segment h of the stretch; K + 1 of them exist
    load_half(x + int64_t(p0) * NC, cur);
    load_half(x + int64_t(2 * p0 + 1) * (NC / 2), na);
    load_half(x + int64_t(min(2 * p0 + 2, K)) * (NC / 2), nb);
#pragma unroll 1
    for (int p = p0; p < p1; ++p) {
      cpx<T> v[16];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const T b = w[r] * T(na[r]);
        v[fft_in_slot<NC, ORD>(r)] = {w[r] * T(cur[r]), b};
        v[fft_in_slot<NC, ORD>(r + 8)] = {T(na[r]) - b, T(nb[r]) - w[r] * T(nb[r])};
        cur[r] = nb[r];
      }
      if (2 * p + 1 >= K) {  // a single segment: zero imaginary part
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r].y = T(0);
      }
      const int pn = min(p + 1, p1 - 1);
      auto next = [&]() {
        load_half(x + int64_t(2 * pn + 1) * (NC / 2), na);
        load_half(x + int64_t(min(2 * pn + 2, K)) * (NC / 2), nb);
      };
      if constexpr (!kLate) next();
      lds_barrier();  // the previous transform's last reads are done
      block_fft<T, NC, -1, false, ORD>(v, sre, sim, t, tw, next);
      add_power(v, p);
    }
  }

  // One-sided sums (Sum) of bins k = t, t + NT, ... in [0, L/2] handed to
  // store(k, sum).
  template <class F> __device__ __forceinline__ void fold(F store) {
    lds_barrier();
    Sum* f = reinterpret_cast<Sum*>(sre);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int i = fft_out_index<NC, ORD>(t, e);
      if constexpr (kPair) f[i] = Sum{tot[e], run[e]};
      else if constexpr (kWide) f[i] = tot[e];
      else f[i] = tot[e] + ACC(run[e]);
    }
    lds_barrier();
    for (int k = t; k <= NC / 2; k += NT) {
      const ACC half = (k == 0 || k == NC / 2) ? ACC(0.5) : ACC(1);
      store(k, sum_scale(sum_add(f[k], f[(NC - k) & (NC - 1)]), half));
    }
  }
};

// Welch PSD of one stretch.  active false: compute but store nothing.
template <class T, class ACC, int NC, int ORD>
__device__ __forceinline__ void welch_item(int K, double norm, int t, const float* x, float* out, const T* tab, T* sre,
                                           T* sim, bool active) {
  WelchItem<T, ACC, NC, ORD> w(tab, t, sre, sim);
  w.pairs(x, K, 0, (K + 1) / 2);
  w.fold([&](int k, auto s) {
    if (active) out[k] = float(sum_value(s) * ACC(norm));
  });
}

// A Welch launch in which workgroup w of G takes the segment pairs
// [start(w), start(w + 1)) of all items' pairs laid end to end, so that every
// workgroup has the same share whatever the number of items.  An item that one
// workgroup holds whole is stored at once; of one that is cut, each piece's
// sums go to a slot of the launch's own, and k_welch_sum adds the slots in
// order.  (The sums are exact, see above: where an item is cut does not change
// its PSD.)
struct WelchCut {
  int G, q, r;   // workgroups; pairs = q G + r
  int np;        // pairs of an item
  // one item per workgroup: nothing is cut (G np may exceed 32 bits then)
  __host__ __device__ bool whole() const { return q == np && r == 0; }
  __device__ __forceinline__ int start(int w) const { return w * q + int(uint32_t(w) * uint32_t(r) / uint32_t(G)); }
  // the last workgroup that starts before pair x
  __device__ __forceinline__ int before(int x) const {
    // ceil(x G / total) - 1; x G < 2^53 is exact, and a quotient below 2^20 that
    // is no whole number is at least 2^-31 from one (total < 2^31)
    return int(ceil(double(x) * double(G) / (double(q) * double(G) + double(r)))) - 1;
  }
};

// A stretch to sum: its first sample, segments and segment pairs.
struct WelchStretch {
  const float* x;
  int K, np;
};

// Runs a workgroup's `left` pairs from pair p0 of `item` on: stretch(item)
// gives the item, whole(item, k, sum) and piece(n, item, k, sum) take bin k's
// one-sided sum of a whole item and of a piece (n = 0: of the first item, 1: of
// the last).
template <class T, class ACC, int NC, int ORD, class Stretch, class Whole, class Piece>
__device__ __forceinline__ void welch_pieces(int item, int p0, int left, int t, const T* tab, T* sre, T* sim,
                                             Stretch stretch, Whole whole, Piece piece) {
  WelchItem<T, ACC, NC, ORD> wi(tab, t, sre, sim);
  const int first = item;
#pragma unroll 1
  while (left > 0) {
    const WelchStretch st = stretch(item);
    const int p1 = min(st.np, p0 + left);
    wi.pairs(st.x, st.K, p0, p1);
    if (p1 - p0 == st.np) wi.fold([&](int k, auto s) { whole(item, k, s); });
    else wi.fold([&](int k, auto s) { piece(item == first ? 0 : 1, item, k, s); });
    left -= p1 - p0;
    p0 = 0;
    ++item;
  }
}

// The slots of cut item `item`, in order, are n of them from workgroup w on:
// slot(w, 0), then slot 2 v of the following workgroups v.
struct WelchSlots {
  int w, n, first;
  __device__ __forceinline__ int64_t slot(int i) const { return i == 0 ? first : 2 * int64_t(w + i); }
};
// (w: the last workgroup that starts at or before the item)
__device__ __forceinline__ WelchSlots welch_slots(const WelchCut& cut, int w, int item) {
  return WelchSlots{w, cut.before((item + 1) * cut.np) - w + 1, 2 * w + (cut.start(w) / cut.np == item ? 0 : 1)};
}

}  // namespace gw
