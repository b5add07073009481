// Device-side physics of the generator: counter-based prior draws, the
// per-sample waveform constants, the per-bin waveform phase and amplitude,
// and the detector response.
//
// Waveform models (section 3.1 of the AMPLFI paper uses an aligned-spin
// IMR model whose inspiral is TaylorF2 to 3.5PN order):
//   approximant 0 -- TaylorF2, 3.5PN phase with 1.5PN spin-orbit and 2PN
//     spin1-spin2 terms, Newtonian amplitude, cut at the Schwarzschild ISCO;
//   approximant 1 -- closed-form inspiral-merger-ringdown: TaylorF2 below
//     f_t = f_RD/2, above it b0 + b1 f + atan((f - f_RD)/f_damp) joined with
//     value and slope continuity; power-law then Lorentzian amplitude; ringdown
//     from the remnant (aligned-spin final-spin fit, radiated-energy fit,
//     fundamental l=m=2 quasi-normal-mode fit); cut at f = 0.2/M.
// The phase is evaluated in revolutions; precision mode 1 and 2 keep it in
// binary64 and reduce it modulo one before a binary32 (mode 1) or binary64
// (mode 2) sine/cosine.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gw {

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// frac(x) in [0, 1)
__device__ __forceinline__ float frac1(float x) { return __builtin_amdgcn_fractf(x); }
__device__ __forceinline__ double frac1(double x) { return __builtin_amdgcn_fract(x); }
// frac(a b), in binary32 of the exact product (within a rounding of [0, 1)):
// rounded first, a product of some thousand revolutions has lost 12 of its
// fraction's bits
__device__ __forceinline__ float frac_product(float a, float b) { return fma_t(a, b, -floorf(a * b)); }
__device__ __forceinline__ double frac_product(double a, double b) { return frac1(a * b); }

// precision-generic math
__device__ __forceinline__ void sincospi_t(float x, float* s, float* c) { sincospif(x, s, c); }
// sin and cos of 2 pi x for x already reduced to [0, 1): the hardware
// sine/cosine take revolutions (max abs error 1.3e-7 measured on gfx950 over
// [0, 1)); binary64 uses the library routine
__device__ __forceinline__ void sincos_rev(float x, float* s, float* c) {
  *s = __builtin_amdgcn_sinf(x);
  *c = __builtin_amdgcn_cosf(x);
}
__device__ __forceinline__ void sincos_rev(double x, double* s, double* c) { sincospi(2.0 * x, s, c); }
__device__ __forceinline__ void sincospi_t(double x, double* s, double* c) { sincospi(x, s, c); }
__device__ __forceinline__ float rsqrt_t(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsqrt_t(double x) { return 1.0 / sqrt(x); }
// reciprocals: binary32 hardware approximation (about 1 ulp); binary64
// hardware seed refined by two Newton steps to full precision
__device__ __forceinline__ float rcp_t(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_t(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return r;
}

constexpr double kPi = 3.14159265358979323846;
constexpr double kMsunSec = 4.925490947641267e-6;                 // G Msun / c^3
constexpr double kMpcSec = 3.085677581491367e22 / 299792458.0;    // Mpc / c
constexpr double kClight = 299792458.0;
constexpr double kStrainScale = 1180591620717411303424.0;         // 2^70
constexpr double kGammaE = 0.5772156649015329;

struct DetGeom {
  double D[6];  // detector tensor xx, xy, xz, yy, yz, zz
  double r[3];  // vertex [m], Earth-fixed
};

struct DevCfg {
  int n_det, N, F, P, L, S, K, Fw, ratio, log2_ratio, approximant, precision, kmin;
  int ord_win, ord_welch;  // FFT radix order of the window and Welch kernels (0: small radix last)
  int occ_welch;           // waves per SIMD the Welch kernel is compiled for (2 or 3)
  double fs, T, invT, f_min, inv_ratio;
  double mc[2], q[2], chi[2], dl[2];
  double f0r[2], Qr[2], hrssr[2];  // sine-Gaussian prior ranges (approximant 2)
  DetGeom det[4];
};

// ---------------------------------------------------------------- Philox
struct U4 { uint32_t a, b, c, d; };

__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint32_t lo0 = 0xD2511F53u * c.a, hi0 = __umulhi(0xD2511F53u, c.a);
    const uint32_t lo1 = 0xCD9E8D57u * c.c, hi1 = __umulhi(0xCD9E8D57u, c.c);
    c = U4{hi1 ^ c.b ^ k0, lo1, hi0 ^ c.d ^ k1, lo0};
  }
  return c;
}

// binary64 uniform in (0, 1) from the first two words
__device__ __forceinline__ double philox_uniform(uint64_t seed, uint64_t index, uint32_t stream,
                                                 uint32_t sub = 0u) {
  U4 o = philox4x32_10(U4{uint32_t(index), uint32_t(index >> 32), stream, sub},
                       uint32_t(seed), uint32_t(seed >> 32));
  return (double(o.a >> 5) * 67108864.0 + double(o.b >> 6) + 0.5) * 0x1p-53;
}

// ------------------------------------------------------- waveform constants
// What a sample's bins need (bin_polar), kept per sample in the workspace.  In
// terms of x = k^(1/3), l = ln(k)/3, the phase in revolutions is
// below f_t  pconst + k^(-5/3) (cN + x^2 (c2 + x (c3 + x (c4 + x ((c5 + b5 l) + x ((c6 + b6x l) + x c7)))))),
// above      mr_p0 + mr_p1 k + atan(X)/(2 pi), X = mr_x0 + mr_x1 k, amplitude Ard / (1 + X^2) beyond f_RD
struct WfScalars {
  double lnv1;          // ln v at bin 1
  double cN;            // Newtonian phase in revolutions at bin k: cN k^(-5/3)
  double c2, c3, c4, c5, b5, c6, b6x, c7;
  double pconst;        // (-phi_c - pi/4) / (2 pi)
  double A0T;           // amplitude A(f_k) = A0T k^(-7/6)
  double mr_p0, mr_p1, mr_x0, mr_x1;
  double Apl, Ard;      // power-law amplitude Apl k^(-2/3) between f_t and f_RD, amplitude at f_RD
  // sine-Gaussian (approximant 2): G(x) = sg_G0 exp(-sg_pt2 x^2), phase phi0 / (2 pi)
  double sg_f0, sg_pt2, sg_G0, sg_rphi;
  double cosi, tc;
  int kend, kt, krd;    // band end; first bins with f >= f_t and f >= f_RD
  int cut_nyquist;
};
// A batch's workspace holds them, and one of the size it had with 280 bytes a
// sample has to be enough.
static_assert(sizeof(WfScalars) <= 280, "workspaces of earlier sizes are accepted");

// The same model at any frequency (the surrogate's targets).
struct WfModel {
  double a[8], b5, b6;  // phase in revolutions below f_t: sum (a_k + b_k ln v) v^(k-5)
  double mr_b0, mr_b1;  // above: b0 + b1 f + atan((f - f_rd) / f_damp)/(2 pi)
  double f_rd, inv_fdamp, fdamp2, ft, At, Ard;
};

// first bin k in [0, kmax] with k/T >= f (k/T formed by a correctly rounded
// division, as the binary64 grid f_k = k/T is formed)
__device__ __forceinline__ int first_bin_at_or_above(double f, double T, int kmax) {
  double x = f * T;
  if (!(x > 0.0)) return 0;
  if (x >= double(kmax)) return kmax;
  int k = int(ceil(x));
  while (k > 0 && double(k - 1) / T >= f) --k;
  while (k < kmax && double(k) / T < f) ++k;
  return k;
}

__device__ __forceinline__ void pn_coefficients(double eta, double q, double chi1, double chi2,
                                                double* c, double* lg) {
  const double dm = (1.0 - q) / (1.0 + q);
  const double chis = 0.5 * (chi1 + chi2), chia = 0.5 * (chi1 - chi2);
  const double pi = kPi;
#pragma unroll
  for (int k = 0; k < 8; ++k) { c[k] = 0.0; lg[k] = 0.0; }
  c[0] = 1.0;
  c[2] = 3715.0 / 756.0 + 55.0 * eta / 9.0;
  c[3] = -16.0 * pi + (113.0 / 3.0) * dm * chia + (113.0 / 3.0 - 76.0 * eta / 3.0) * chis;
  c[4] = 15293365.0 / 508032.0 + 27145.0 * eta / 504.0 + 3085.0 * eta * eta / 72.0
         - (395.0 / 4.0) * eta * chi1 * chi2;
  const double p5 = pi * (38645.0 / 756.0 - 65.0 * eta / 9.0);
  // psi5 (1 + 3 ln(v / v_lso)), v_lso = 6^(-1/2):  ln v_lso = -ln(6)/2
  c[5] = p5 * (1.0 + 1.5 * log(6.0));
  lg[5] = 3.0 * p5;
  const double c6 = 11583231236531.0 / 4694215680.0 - 640.0 * pi * pi / 3.0
                    - (6848.0 / 21.0) * kGammaE
                    + (-15737765635.0 / 3048192.0 + 2255.0 * pi * pi / 12.0) * eta
                    + 76055.0 * eta * eta / 1728.0 - 127825.0 * eta * eta * eta / 1296.0;
  c[6] = c6 - (6848.0 / 21.0) * log(4.0);
  lg[6] = -(6848.0 / 21.0);
  c[7] = pi * (77096675.0 / 254016.0 + 378515.0 * eta / 1512.0 - 74045.0 * eta * eta / 756.0);
}

// The per-sample set-up runs in groups of kSetupLanes consecutive lanes of a
// wavefront that hold the same sample: every lane does the cheap arithmetic,
// and the powers, roots, logarithms and sines, which are what the set-up's
// latency is made of, are evaluated one per lane and exchanged.  One thread
// per sample took 25 us for a single sample, a chain of 27 pow() calls.
constexpr int kSetupLanes = 16;
__device__ __forceinline__ double lane_value(double v, int lane) { return __shfl(v, lane, kSetupLanes); }
__device__ __forceinline__ int lane_value(int v, int lane) { return __shfl(v, lane, kSetupLanes); }

// TaylorF2 intrinsic phase P(f) [rad] and dP/df at v = (pi M f)^(1/3), full binary64
__device__ __forceinline__ void tf2_phase_and_slope(double f, double v, double lnv, double eta, const double* c,
                                                    const double* lg, double* P, double* dP) {
  const double iv = 1.0 / v, iv2 = iv * iv;
  double vk = iv2 * iv2 * iv;  // v^(k-5)
  double s = 0.0, ds = 0.0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const double ck = c[k] + lg[k] * lnv;
    s += ck * vk;
    ds += ((k - 5) * ck + lg[k]) * (vk * iv);
    vk *= v;
  }
  const double pre = 3.0 / (128.0 * eta);
  *P = pre * s;
  *dP = pre * ds * v / (3.0 * f);
}

// Sines and cosines of the sky angles.
struct SkyAngles { double sr, cr, sd, cd, sp, cp; };

// Waveform constants of one sample from its parameter rows p[0..10] (held by
// every lane of the group; lane = this lane's place in it).  All lanes return
// the same values.
__device__ __forceinline__ void wf_setup(const double* p, const DevCfg& cf, int lane, WfScalars& w, WfModel& m,
                                         SkyAngles& sky) {
  // iota, RA, dec, psi: one sine and cosine per lane
  // (selected as values: a selected element's address would keep p in memory)
  const double iota = p[5], ra = p[6], dec = p[7], psi = p[8];
  const double ang = lane == 0 ? iota : lane == 1 ? ra : lane == 2 ? dec : psi;
  double sn, cs;
  sincos(ang, &sn, &cs);
  w.cosi = lane_value(cs, 0);
  sky = {lane_value(sn, 1), lane_value(cs, 1), lane_value(sn, 2), lane_value(cs, 2), lane_value(sn, 3), lane_value(cs, 3)};
  w.tc = p[10];
  if (cf.approximant == 2) {
    // sine-Gaussian: rows 0 f0, 1 Q, 2 hrss, 5 iota, 9 phi0, 10 t0
    const double f0 = p[0], Q = p[1], hrss = p[2];
    const double tau = Q / (sqrt(2.0) * kPi * f0);
    const double A = kStrainScale * hrss / sqrt(tau * sqrt(0.5 * kPi));
    w.sg_f0 = f0;
    w.sg_pt2 = kPi * kPi * tau * tau;
    w.sg_G0 = A * 0.5 * sqrt(kPi) * tau;
    w.sg_rphi = p[9] / (2.0 * kPi);
    w.kend = cf.N / 2;
    w.kt = w.krd = w.kend;
    w.cut_nyquist = f0 + 5.0 / (kPi * tau) >= 0.5 * cf.fs ? 1 : 0;
    return;
  }
  const double mc = p[0], q = p[1], chi1 = p[2], chi2 = p[3], dl = p[4], phic = p[9];
  const double eta = q / ((1.0 + q) * (1.0 + q));
  // remnant: aligned-spin final-spin fit, non-spinning radiated-energy fit
  const double a_tot = (chi1 + chi2 * q * q) / (1.0 + q * q);
  double af = a_tot - 0.1229 * a_tot * a_tot * eta + 0.4537 * a_tot * eta * eta
              - 2.8904 * a_tot * eta + 2.0 * sqrt(3.0) * eta - 3.5171 * eta * eta
              + 2.5763 * eta * eta * eta;
  af = fmin(fmax(af, -0.99), 0.99);
  const double px = lane == 0 ? eta : lane == 1 ? mc * kMsunSec : lane == 2 ? cf.T : 1.0 - af;
  const double py = lane == 0 ? -0.6 : lane == 1 ? 5.0 / 6.0 : lane == 2 ? 7.0 / 6.0 : lane == 3 ? 0.1292 : -0.4990;
  const double pw = pow(px, py);
  const double Ms = mc * lane_value(pw, 0) * kMsunSec;
  double c[8], lg[8];
  pn_coefficients(eta, q, chi1, chi2, c, lg);
  const double rev = 3.0 / (128.0 * eta) / (2.0 * kPi);
#pragma unroll
  for (int k = 0; k < 8; ++k) m.a[k] = rev * c[k];
  m.b5 = w.b5 = rev * lg[5];
  m.b6 = rev * lg[6];
  w.pconst = (-phic - 0.25 * kPi) / (2.0 * kPi);
  const double A0 = kStrainScale * sqrt(5.0 / 24.0) * pow(kPi, -2.0 / 3.0) * lane_value(pw, 1) / (dl * kMpcSec);
  w.A0T = A0 * lane_value(pw, 2);
  const int knyq = cf.N / 2;
  double f_cut, f_t = 1.0, f_rd = 1.0, f_damp = 1.0;
  if (cf.approximant == 0) {
    f_cut = 1.0 / (pow(6.0, 1.5) * kPi * Ms);
  } else {
    f_cut = 0.2 / Ms;
    const double erad = 0.0559745 * eta + 0.580951 * eta * eta - 0.960673 * eta * eta * eta
                        + 3.35241 * eta * eta * eta * eta;
    const double Mf = Ms * (1.0 - erad);
    const double omega = 1.5251 - 1.1568 * lane_value(pw, 3);
    const double Q = 0.7 + 1.4187 * lane_value(pw, 4);
    f_rd = omega / (2.0 * kPi * Mf);
    f_damp = f_rd / (2.0 * Q);
    f_t = 0.5 * f_rd;
  }
  // v and ln v at bin 1 (lane 0) and at f_t; the band edges one per lane
  const double v = cbrt(kPi * Ms * (lane == 0 ? cf.invT : f_t)), lnv = log(v);
  const int kb = first_bin_at_or_above(lane == 0 ? f_cut : lane == 1 ? f_t : f_rd, cf.T, knyq);
  const double v1 = lane_value(v, 0);
  w.lnv1 = lane_value(lnv, 0);
  w.cN = m.a[0] / (v1 * v1 * v1 * v1 * v1);
  w.kend = lane_value(kb, 0);
  w.cut_nyquist = f_cut > 0.5 * cf.fs ? 1 : 0;
  {
    const double iv = 1.0 / v1, iv2 = iv * iv;
    w.c2 = m.a[2] * iv2 * iv;
    w.c3 = m.a[3] * iv2;
    w.c4 = m.a[4] * iv;
    w.c5 = m.a[5] + w.b5 * w.lnv1;
    w.c6 = (m.a[6] + m.b6 * w.lnv1) * v1;
    w.b6x = m.b6 * v1;
    w.c7 = m.a[7] * v1 * v1;
  }
  if (cf.approximant == 0) {
    w.mr_p0 = w.mr_p1 = w.mr_x0 = w.mr_x1 = 0.0;
    w.kt = w.kend;
    w.krd = w.kend;
    w.Ard = w.Apl = 0.0;
    return;
  }
  double Pt, dPt;
  tf2_phase_and_slope(f_t, lane_value(v, 1), lane_value(lnv, 1), eta, c, lg, &Pt, &dPt);
  const double x_t = (f_t - f_rd) / f_damp;
  const double b1 = dPt - (1.0 / f_damp) / (1.0 + x_t * x_t);
  const double b0 = Pt - b1 * f_t - atan(x_t);
  m.mr_b0 = b0 / (2.0 * kPi);
  m.mr_b1 = b1 / (2.0 * kPi);
  m.f_rd = f_rd;
  m.inv_fdamp = 1.0 / f_damp;
  w.mr_p0 = m.mr_b0 + w.pconst;
  w.mr_p1 = m.mr_b1 * cf.invT;
  w.mr_x0 = -f_rd * m.inv_fdamp;
  w.mr_x1 = cf.invT * m.inv_fdamp;
  const double pw2 = pow(lane == 0 ? f_t : lane == 1 ? f_rd / f_t : f_t * cf.T,
                         lane == 0 ? -7.0 / 6.0 : lane == 1 ? -2.0 / 3.0 : 2.0 / 3.0);
  m.At = A0 * lane_value(pw2, 0);
  m.Ard = w.Ard = m.At * lane_value(pw2, 1);
  m.ft = f_t;
  m.fdamp2 = f_damp * f_damp;
  w.Apl = m.At * lane_value(pw2, 2);
  w.kt = min(lane_value(kb, 1), w.kend);
  w.krd = min(lane_value(kb, 2), w.kend);
}

// The same for column b of params [11 or 12][B], by the first kSetupLanes
// threads of a workgroup (thread t of them); lane 0 writes w, or the model m.
__device__ __forceinline__ void wf_setup_column(const double* __restrict__ params, int64_t B, int64_t b,
                                                const DevCfg& cf, int t, WfScalars* w, WfModel* m = nullptr) {
  const double mine = params[min(t, 10) * B + b];
  double p[11];
#pragma unroll
  for (int r = 0; r < 11; ++r) p[r] = lane_value(mine, r);
  WfScalars v = {};
  WfModel vm = {};
  SkyAngles sky;
  wf_setup(p, cf, t, v, vm, sky);
  if (t != 0) return;
  if (w) *w = v;
  if (m) *m = vm;
}

// Powers of a bin number.
struct BinPowers { double kc, lk, k53; };  // k^(1/3), ln(k)/3, k^(-5/3)

// Waveform phase in revolutions (phi_c included, without the time shift) and
// amplitude (type T) at bin k.  TP is binary64 for precision modes 1 and 2 and
// binary32 for mode 0; FULL selects a binary64 arctangent for the (bounded)
// ringdown term (mode 2).  The amplitude is A0T k^(-7/6) = A0T k^(-5/3) k^(1/2)
// below f_t, At (f/f_t)^(-2/3) = Apl k^(-2/3) up to f_RD, then the Lorentzian.
// Twelve binary64 operations below f_t; with the coefficients in terms of v and
// 1/v from a reciprocal there were 28.
template <class T, class TP, bool FULL>
__device__ __forceinline__ void bin_polar(const WfScalars& w, int k, const BinPowers& t, TP* rev, T* amp) {
  if (k < w.kt) {
    const TP x = TP(t.kc), l = TP(t.lk);
    TP p = fma_t(x, TP(w.c7), fma_t(TP(w.b6x), l, TP(w.c6)));
    p = fma_t(x, p, fma_t(TP(w.b5), l, TP(w.c5)));
    p = fma_t(x, p, TP(w.c4));
    p = fma_t(x, p, TP(w.c3));
    p = fma_t(x, p, TP(w.c2));
    p = fma_t(x * x, p, TP(w.cN));
    *rev = fma_t(p, TP(t.k53), TP(w.pconst));
    const T kf = T(k);
    *amp = T(w.A0T) * T(t.k53) * (kf * rsqrt_t(kf));
    return;
  }
  const double x = fma_t(double(k), w.mr_x1, w.mr_x0);
  const TP lin = fma_t(TP(k), TP(w.mr_p1), TP(w.mr_p0));
  if constexpr (FULL) *rev = lin + TP(atan(x) * (1.0 / (2.0 * kPi)));
  else *rev = lin + TP(atanf(float(x)) * float(1.0 / (2.0 * kPi)));
  if (k < w.krd) {
    const T kc = T(t.kc);
    *amp = T(w.Apl) * rcp_t(kc * kc);
  } else {
    const T xx = T(x);
    *amp = T(w.Ard) * rcp_t(fma_t(xx, xx, T(1)));
  }
}

// -------------------------------------------------------- detector response
struct DetScalars { double fp, fx, tau; };

__device__ __forceinline__ DetScalars det_response(const DetGeom& g, const SkyAngles& a, double tc) {
  const double sr = a.sr, cr = a.cr, sd = a.sd, cd = a.cd, sp = a.sp, cp = a.cp;
  const double et[3] = {sd * cr, sd * sr, -cd};
  const double ep[3] = {-sr, cr, 0.0};
  double p[3], qv[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    p[i] = cp * et[i] + sp * ep[i];
    qv[i] = -sp * et[i] + cp * ep[i];
  }
  const double* D = g.D;
  const double Dm[3][3] = {{D[0], D[1], D[2]}, {D[1], D[3], D[4]}, {D[2], D[4], D[5]}};
  double fp = 0.0, fx = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      fp += Dm[i][j] * (p[i] * p[j] - qv[i] * qv[j]);
      fx += Dm[i][j] * (p[i] * qv[j] + qv[i] * p[j]);
    }
  const double n[3] = {cd * cr, cd * sr, sd};
  const double dt = -(n[0] * g.r[0] + n[1] * g.r[1] + n[2] * g.r[2]) / kClight;
  return DetScalars{fp, fx, tc + dt};
}

}  // namespace gw
