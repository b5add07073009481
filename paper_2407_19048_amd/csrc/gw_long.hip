// Long windows (N > 32768 samples, e.g. long-duration binary-neutron-star
// signals): the half-length complex transform of NC = N/2 points no longer
// fits in one workgroup's LDS and runs as a four-step FFT through HBM, with
// NC = N1 x N2, N1 the row length (one workgroup transform in LDS) and
// N2 = NC/N1 in {4, 8, 16, 32} (in registers).  N1 = 8192 up to N = 2^19
// (two workgroups of 512 threads share a CU), 16384 for N = 2^20 (N2 = 32).
// With c[m] = y[2m] + i y[2m+1]:
//
//   forward  columns  w[k2][m1] = W_NC^(m1 k2) sum_m2 c[m1 + N1 m2] W_N2^(m2 k2)
//            rows     X[k2 + N2 k1] = sum_m1 w[k2][m1] W_N1^(m1 k1)   (in place)
//   bins     real-spectrum unpack of the pair (k, NC - k), in-register
//            signal, whitening, repack for the inverse (in place, on the
//            transposed layout X'[k2][k1] = X[k2 + N2 k1])
//   inverse  rows     u[k2][m1] = sum_k1 Z[k2 + N2 k1] W_N1^(-m1 k1)  (in place)
//            columns  c[m1 + N1 m2] = (1/NC) sum_k2 W_N2^(-m2 k2) W_NC^(-m1 k2) u[k2][m1]
//
// The thread of column m1 reads u[k2][m1] for every k2 and writes
// c[m1 + N1 m2] for every m2: the same complex positions, so the inverse
// also runs in place.  Every pass works inside the caller's output buffer
// (N floats = NC complex per window); no other memory is needed.
#include <hip/hip_runtime.h>

#include <string>

#include "gw_fft.hpp"
#include "gw_physics.hpp"
#include "gw_internal.hpp"
#include "gw_items.hpp"
#include "../../include/gwgen.h"

using namespace gw;

namespace {

// Waves per SIMD the row kernels are compiled for: two 512-thread workgroups
// (N1 = 8192) or one 1024-thread workgroup (N1 = 16384) per CU, 128 VGPRs.
constexpr int kRowWaves = 4;

// In-register DFT of length R (natural order in and out), DIR = -1 forward.
template <int R, int DIR, class T>
__device__ __forceinline__ void dft_small(cpx<T>* a) {
  if constexpr (R == 2) dft2<DIR>(a);
  else if constexpr (R == 4) dft4<DIR>(a);
  else if constexpr (R == 8) dft8<DIR>(a);
  else if constexpr (R == 16) dft16<DIR>(a);
  else {
    static_assert(R == 32, "N2 in {4, 8, 16, 32}");
    cpx<T> e[16], o[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      e[i] = a[2 * i];
      o[i] = a[2 * i + 1];
    }
    dft16<DIR>(e);
    dft16<DIR>(o);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      T s, c;
      sincospi_t(T(2 * k) / T(32), &s, &c);  // exp(DIR 2 pi i k / 32)
      const cpx<T> w = {c, T(DIR) * s};
      const cpx<T> t = cmul(o[k], w);
      a[k] = cadd(e[k], t);
      a[k + 16] = csub(e[k], t);
    }
  }
}

// Powers of bin k from its table entry: k^(1/3) = k^(-5/3) k^2.  (The power
// -5/3 from a table of k^(1/3) took a binary64 reciprocal, 14 of the 220
// instructions of a bin; in the kernels of short windows, which read k^(1/3)
// as well, two tables instead of three changed nothing.)
__device__ __forceinline__ BinPowers bin_powers(int k, BinTab t) {
  const double kd = double(k);
  return {t.k53 * (kd * kd), t.lk, t.k53};
}

struct LongArgs {
  WinArgs w;           // cf, tables, per-sample data, psd, status; out = the in-place buffer
  const void* twc;     // cpx<float>[N2][N1]: exp(-2 pi i m1 k2 / NC) at [k2][m1]
  const void* twr;     // cpx<float>[NC/2 + 1]: exp(-2 pi i k / N)
  const void* tw1;     // pass twiddle tables of the N1-point transform
  const float* x;      // real input of the forward columns (strain rows or the background)
  int NC, N2, l2n2;    // NC = N1 N2, l2n2 = log2(N2)
  // bin tables in the transposed layout (bin k at (k mod N2) N1 + k / N2):
  const BinTab* bins_t;
  const cpx<float>* twr_t;   // exp(-2 pi i k / N)
};

// x row of window item bd (SRC 0: strain [B][D][N]; SRC 1, 2: background at o + P)
template <int SRC>
__device__ __forceinline__ const float* long_input(const LongArgs& a, int64_t bd) {
  const DevCfg& cf = a.w.cf;
  const int64_t b = bd / cf.n_det;
  const int d = int(bd - b * cf.n_det);
  if constexpr (SRC == 0) return a.x + bd * int64_t(cf.N);
  else return a.x + int64_t(d) * a.w.L_bg + load_const(a.w.offset + b) + cf.P;
}

// Forward columns: one thread per column m1, grid (N1/256, B*D).
template <int N1, int N2, int SRC>
__global__ __launch_bounds__(256) void k_long_cols_fwd(LongArgs a) {
  const int m1 = blockIdx.x * 256 + threadIdx.x;
  const int64_t bd = blockIdx.y;
  const float* x = long_input<SRC>(a, bd);
  float2* buf = reinterpret_cast<float2*>(a.w.out) + bd * a.NC;
  const cpx<float>* twc = reinterpret_cast<const cpx<float>*>(a.twc);
  cpx<float> v[N2];
#pragma unroll
  for (int m2 = 0; m2 < N2; ++m2) {
    float2 q;
    __builtin_memcpy(&q, x + 2 * (int64_t(m1) + int64_t(N1) * m2), sizeof(q));
    v[m2] = {q.x, q.y};
  }
  dft_small<N2, -1>(v);
#pragma unroll
  for (int k2 = 0; k2 < N2; ++k2) {
    const cpx<float> w = k2 ? cmul(v[k2], twc[k2 * N1 + m1]) : v[k2];
    buf[int64_t(k2) * N1 + m1] = {w.x, w.y};
  }
}

// Inverse columns: twiddle, inverse DFT over k2, scale, store real samples in
// place; SRC 2 adds the noise window.
template <int N1, int N2, int SRC>
__global__ __launch_bounds__(256) void k_long_cols_inv(LongArgs a) {
  const int m1 = blockIdx.x * 256 + threadIdx.x;
  const int64_t bd = blockIdx.y;
  float2* buf = reinterpret_cast<float2*>(a.w.out) + bd * a.NC;
  const cpx<float>* twc = reinterpret_cast<const cpx<float>*>(a.twc);
  cpx<float> v[N2];
#pragma unroll
  for (int k2 = 0; k2 < N2; ++k2) {
    const float2 q = buf[int64_t(k2) * N1 + m1];
    const cpx<float> u = {q.x, q.y};
    v[k2] = k2 ? twmul<+1>(u, twc[k2 * N1 + m1]) : u;
  }
  dft_small<N2, +1>(v);
  const float sc = SRC == 2 ? 0.5f / float(a.NC) : whitened_scale<float>(a.NC);
  const float* nz = nullptr;
  if constexpr (SRC == 2) nz = long_input<2>(a, bd);
#pragma unroll
  for (int m2 = 0; m2 < N2; ++m2) {
    const int64_t m = int64_t(m1) + int64_t(N1) * m2;
    float2 y = {v[m2].x * sc, v[m2].y * sc};
    if constexpr (SRC == 2) {
      y.x += nz[2 * m];
      y.y += nz[2 * m + 1];
    }
    buf[m] = y;
  }
}

// Row transforms of length N1 in place: grid B*D*N2 workgroups of N1/16.
template <int N1, int DIR>
__global__ __launch_bounds__(N1 / 16, kRowWaves) void k_long_rows(LongArgs a) {
  constexpr int NT = N1 / 16, LS = LdsSize<N1>::value;
  __shared__ float lds[2 * LS];
  const int t = threadIdx.x;
  float2* row = reinterpret_cast<float2*>(a.w.out) + int64_t(blockIdx.x) * N1;
  PassTwiddle<float, N1, 0> tw{reinterpret_cast<const cpx<float>*>(a.tw1)};
  cpx<float> v[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const float2 q = row[t + NT * j];
    v[fft_in_slot<N1, 0>(j)] = {q.x, q.y};
  }
  block_fft<float, N1, DIR, false, 0>(v, lds, lds + LS, t, tw);
#pragma unroll
  for (int e = 0; e < 16; ++e) row[fft_out_index<N1, 0>(t, e)] = {v[e].x, v[e].y};
}

// Inject: pack the given projected spectrum for the inverse transform, one
// thread per pair (k, NC - k), k in [0, NC/2], reading hdet by k:
// grid (ceil((NC/2 + 1)/256), B*D).  The packed pair lands at its place in
// the transposed layout X'[k2][k1] = X[k2 + N2 k1] of the inverse rows.
template <int N1>
__global__ __launch_bounds__(256) void k_long_inject(LongArgs a, const float* hdet) {
  const int64_t bd = blockIdx.y;
  const int NC = a.NC, N2 = a.N2;
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k > NC / 2) return;
  float2* buf = reinterpret_cast<float2*>(a.w.out) + bd * NC;
  const int km = NC - k;
  auto pos = [&](int kk) { kk &= NC - 1; return int64_t(kk & (N2 - 1)) * N1 + (kk >> a.l2n2); };
  const cpx<float> W = reinterpret_cast<const cpx<float>*>(a.twr)[k];  // exp(-2 pi i k / N)
  const float2* h = reinterpret_cast<const float2*>(hdet) + bd * (NC + 1);
  const float2 h0 = h[k], h1 = h[km];
  // irfft ignores Im at DC and Nyquist
  const cpx<float> Yk = {h0.x, k == 0 ? 0.f : h0.y};
  const cpx<float> Ym = {h1.x, k == 0 ? 0.f : h1.y};
  cpx<float> zk, zm;
  repack_pair(Yk, 1.f, Ym, 1.f, W, &zk, &zm);
  buf[pos(k)] = {zk.x, zk.y};
  if (k != 0 && km != k) buf[pos(km)] = {zm.x, zm.y};
}

// Global inputs of one pair of packed-spectrum bins (k, km = NC - k),
// k <= NC/2: the real-FFT twiddle exp(-2 pi i k / N), the bin tables of both
// bins (SRC 1) and the PSD values around both bins.  pk, pm: positions of k
// and km in the transposed bin tables.
struct LongPairIn {
  cpx<float> W;
  BinTab b[2];
  PsdAround g;
};

template <int SRC>
__device__ __forceinline__ LongPairIn long_pair_fetch(const LongArgs& a, const float* psd, int k, int64_t pk,
                                                      int64_t pm) {
  LongPairIn in;
  in.W = a.twr_t[pk];
  if constexpr (SRC == 1) {
    in.b[0] = a.bins_t[pk];
    in.b[1] = a.bins_t[pm];
  }
  in.g = psd_around(a.w.cf, psd, k, a.NC);
  return in;
}

// The item's projection (SRC 1).
__device__ __forceinline__ Projection<float> long_projection(const LongArgs& a, const WfScalars& w, int64_t b, int d) {
  const DevCfg& cf = a.w.cf;
  const DetScalars dsh = load_const(a.w.dsc + (b * cf.n_det + d));
  return {float(cf.fs * dsh.fp * (1.0 + w.cosi * w.cosi)), float(2.0 * cf.fs * dsh.fx * w.cosi), dsh.tau * cf.invT};
}

// One pair of packed-spectrum bins (k, km = NC - k), k <= NC/2: A = Z[k] and
// Bm = Z[km] in; out, the packed spectrum of the whitened window (SRC 1 with
// the in-register signal added) at the same two bins, scaled (whitened_scale).
template <class TP, int SRC>
__device__ __forceinline__ void long_pair(const LongArgs& a, const WfScalars& wsh, const Projection<float>& pr,
                                          const LongPairIn& in, int k, cpx<float>& A, cpx<float>& Bm, uint32_t& flag) {
  const DevCfg& cf = a.w.cf;
  const int NC = a.NC, km = NC - k;
  cpx<float> Yk, Ym;
  unpack_pair(A, Bm, in.W, &Yk, &Ym);
  if constexpr (SRC == 1) {
    add_signal<float, TP, false>(cf, wsh, pr, k, [&](int kk) { return bin_powers(kk, in.b[0]); }, &Yk);
    add_signal<float, TP, false>(cf, wsh, pr, km, [&](int kk) { return bin_powers(kk, in.b[1]); }, &Ym);
  }
  float gk, gm;
  psd_gains<float>(cf, in.g, k, NC, flag, &gk, &gm);
  repack_pair(Yk, gk, Ym, gm, in.W, &A, &Bm);
}

// Bins: the real-spectrum unpack of each pair (k, NC - k), k in [0, NC/2],
// then (SRC 1) the in-register signal, the whitening gain and the repack for
// the inverse; SRC 0 whitens only.  Thread (k1, r) takes the element at row
// r, column k1 of X'[k2][k1] = X[k2 + N2 k1], i.e. k = r + N2 k1, or its
// mirror NC - k (row N2 - r, column N1 - 1 - k1) when k > NC/2, so that a
// wavefront reads and writes runs of consecutive (or reversed) columns of two
// rows, and reads the bin tables in the same transposed layout.  Rows 0 and
// N2/2 pair with themselves and use half their columns.  Two pairs per
// thread, columns k1 and k1 + 256 (grid (N1/512, B*D, N2/2 + 1)): both pairs'
// inputs are loaded before either is computed, so the second pair's loads
// overlap the first pair's arithmetic.  Idle lanes load a real pair too (k is
// clamped into range) and only skip their stores.
template <int N1, class TP, int SRC>
__global__ __launch_bounds__(256) void k_long_bins(LongArgs a) {
  static_assert(SRC == 0 || SRC == 1, "whiten or fused");
  constexpr int J = 2;
  const int64_t bd = blockIdx.y;
  const DevCfg& cf = a.w.cf;
  const int NC = a.NC, N2 = a.N2;
  const int r = blockIdx.z;
  const int64_t b = bd / cf.n_det;
  const int d = int(bd - b * cf.n_det);
  float2* buf = reinterpret_cast<float2*>(a.w.out) + bd * NC;
  const float* psd = a.w.psd + bd * cf.Fw;
  auto pos = [&](int kk) { kk &= NC - 1; return int64_t(kk & (N2 - 1)) * N1 + (kk >> a.l2n2); };
  __shared__ uint32_t sflag;
  if (threadIdx.x == 0) sflag = 0u;
  __syncthreads();
  int k[J];
  bool ok[J];
  float2 qa[J], qb[J];
  LongPairIn in[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int k1 = blockIdx.x * (256 * J) + 256 * j + threadIdx.x;  // < N1
    const int kr = r + N2 * k1;
    ok[j] = (r == 0) ? (k1 <= N1 / 2) : (2 * r == N2) ? (k1 < N1 / 2) : true;
    k[j] = min(kr, NC - kr);
    const int64_t pk = pos(k[j]), pm = pos(NC - k[j]);
    qa[j] = buf[pk];
    qb[j] = buf[pm];
    in[j] = long_pair_fetch<SRC>(a, psd, k[j], pk, pm);
  }
  WfScalars wsh;
  Projection<float> pr = {0.f, 0.f, 0.0};
  if constexpr (SRC == 1) {
    wsh = load_const(a.w.wf + b);
    pr = long_projection(a, wsh, b, d);
  }
  uint32_t flag = 0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int kk = k[j], km = NC - kk;
    cpx<float> A = {qa[j].x, qa[j].y}, Bm = {qb[j].x, qb[j].y};
    uint32_t fj = 0;
    long_pair<TP, SRC>(a, wsh, pr, in[j], kk, A, Bm, fj);
    if (ok[j]) {
      buf[pos(kk)] = {A.x, A.y};
      if (kk != 0 && km != kk) buf[pos(km)] = {Bm.x, Bm.y};
      flag |= fj;
    }
  }
  if (flag) atomicOr(&sflag, flag);
  __syncthreads();
  if (threadIdx.x == 0 && sflag && a.w.status) atomicOr(a.w.status + b, sflag);
}

// Rows, bins and inverse rows of two rows in one workgroup (replacing three
// passes through HBM).  Bin k = r + N2 c sits at row r, column c of the
// transposed spectrum, and its partner NC - k at row N2 - r, column N1 - 1 - c
// (row 0 and row N2/2 pair with themselves: columns N1 - c and N1 - 1 - c).
// Grid: B*D*N2/2 workgroups of N1/16 threads; workgroup (item, r) owns rows r
// and N2 - r, workgroup (item, 0) the self-paired rows 0 and N2/2, one after
// the other: all workgroups have two rows to do, so that whole rounds of them
// fill the chip (with the self-paired rows as workgroups of their own, 96
// windows of N2 = 32 took 3.2 rounds of 512 instead of 3).
// Two-row pairs: the spectrum of row r stays in registers (thread t holds the
// columns t + NT j) while row N2 - r is transformed and stored to LDS in
// natural order.  Each thread then pairs its row-r columns with their
// partners read from LDS, keeps row r's results and writes row N2 - r's to
// LDS in place (every LDS word is read and written by one thread only); then
// the inverse transforms of row N2 - r (from LDS) and of row r (from
// registers).  Each row is read and written once, where row r made two more
// round trips through the buffer to save registers.  96 windows of 2^19
// samples: 248 us with both of these as they were, 222 now, of which the
// vector arithmetic takes 120 to 145 and the rows' 400 MB 80 (207 since with
// k^(-5/3) from a table, see bin_powers; 210 with sines in the transforms'
// first stages, see kSineTable).  Rows are left unscaled, as the separate row
// passes leave them.
template <int N1, class TP, int SRC>
__global__ __launch_bounds__(N1 / 16, kRowWaves) void k_long_rowpair(LongArgs a) {
  static_assert(SRC == 0 || SRC == 1, "whiten or fused");
  constexpr int NT = N1 / 16, LS = LdsSize<N1>::value;
  __shared__ float lds[2 * LS];
  __shared__ uint32_t sflag;
  float* sre = lds;
  float* sim = lds + LS;
  const int t = threadIdx.x;
  const DevCfg& cf = a.w.cf;
  const int NC = a.NC, N2 = a.N2;
  const int64_t bd = blockIdx.x / (N2 / 2);
  const int rA = int(blockIdx.x - bd * (N2 / 2));
  const int64_t b = bd / cf.n_det;
  const int d = int(bd - b * cf.n_det);
  float2* buf = reinterpret_cast<float2*>(a.w.out) + bd * NC;
  const float* psd = a.w.psd + bd * cf.Fw;
  const cpx<float>* tw1 = reinterpret_cast<const cpx<float>*>(a.tw1);
  // a fresh table pointer per transform (see opaque)
  auto tw = [&]() { return PassTwiddle<float, N1, 0>{opaque(tw1)}; };
  if (t == 0) sflag = 0u;
  Projection<float> pr = {0.f, 0.f, 0.0};
  WfScalars wsh;
  if constexpr (SRC == 1) {
    wsh = load_const(a.w.wf + b);
    pr = long_projection(a, wsh, b, d);
  }
  uint32_t flag = 0;
  // Each phase below takes its own copy of the lane index and row pointers
  // (fresh_lane, fresh): without them the compiler shares the index and
  // address arithmetic of the transforms and keeps it live throughout,
  // beyond the 128 registers a 1024-thread workgroup allows.
  auto load_row = [&](cpx<float>* v, float2* row) {
    const int tl = fresh_lane(t);
    float2* r = fresh(row);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float2 q = r[tl + NT * j];
      v[fft_in_slot<N1, 0>(j)] = {q.x, q.y};
    }
  };
  auto store_row = [&](const cpx<float>* v, float2* row) {
    const int tl = fresh_lane(t);
    float2* r = fresh(row);
#pragma unroll
    for (int e = 0; e < 16; ++e) r[fft_out_index<N1, 0>(tl, e)] = {v[e].x, v[e].y};
  };
  auto store_lds = [&](const cpx<float>* v) {
    const int tl = fresh_lane(t);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int i = lpad<float>(fft_out_index<N1, 0>(tl, e));
      sre[i] = v[e].x;
      sim[i] = v[e].y;
    }
  };
  if (rA == 0) {
    // self-paired rows (uniform over the workgroup): spectrum to LDS, pairs
    // in LDS, inverse transform from LDS
#pragma unroll 1
    for (int r = 0; r < N2; r += N2 / 2) {
      float2* row = buf + int64_t(r) * N1;
      cpx<float> v[16];
      load_row(v, row);
      if (r) lds_barrier();  // the row before is done with LDS
      block_fft<float, N1, -1, false, 0>(v, sre, sim, fresh_lane(t), tw());
      lds_barrier();
      store_lds(v);
      lds_barrier();
      const int tl = fresh_lane(t);
      // column of iteration j and its mirror; the pair's global inputs are
      // fetched one iteration ahead (clamped to the lower bin, so that every
      // iteration loads a valid pair) to overlap their latency
      auto cols = [&](int j, int& c, int& cm, int& k) {
        c = tl + NT * j;
        cm = r == 0 ? ((N1 - c) & (N1 - 1)) : (N1 - 1 - c);
        k = r + N2 * c;
        if (k > NC - k) {  // the partner's thread handles the pair; fetch it anyway
          const int x = c;
          c = cm;
          cm = x;
          k = NC - k;
        }
      };
      int c, cm, k;
      cols(0, c, cm, k);
      LongPairIn nxt = long_pair_fetch<SRC>(a, psd, k, int64_t(r) * N1 + c, int64_t(r) * N1 + cm);
#pragma unroll 1
      for (int j = 0; j < 16; ++j) {
        const LongPairIn cur = nxt;
        const int cj = c, cmj = cm, kj = k;
        const bool mine = r + N2 * (tl + NT * j) <= NC - (r + N2 * (tl + NT * j));
        if (j + 1 < 16) {
          cols(j + 1, c, cm, k);
          nxt = long_pair_fetch<SRC>(a, psd, k, int64_t(r) * N1 + c, int64_t(r) * N1 + cm);
        }
        if (!mine) continue;  // the partner's thread handles the pair
        const int km = NC - kj;
        const int ic = lpad<float>(cj), im = lpad<float>(cmj);
        cpx<float> A = {sre[ic], sim[ic]}, Bm = {sre[im], sim[im]};
        long_pair<TP, SRC>(a, wsh, pr, cur, kj, A, Bm, flag);
        sre[ic] = A.x;
        sim[ic] = A.y;
        if (kj != 0 && km != kj) {
          sre[im] = Bm.x;
          sim[im] = Bm.y;
        }
      }
      lds_barrier();
      block_fft<float, N1, +1, true, 0>(v, sre, sim, fresh_lane(t), tw());
      store_row(v, row);
    }
  } else {
    const int rB = N2 - rA;
    float2* rowA = buf + int64_t(rA) * N1;
    float2* rowB = buf + int64_t(rB) * N1;
    cpx<float> A[16], v[16];
    load_row(v, rowA);
    block_fft<float, N1, -1, false, 0>(v, sre, sim, fresh_lane(t), tw());
    // A[j]: column t + NT j of row rA
    constexpr int RL = PlanEnds<N1, 0>::RLAST;
#pragma unroll
    for (int e = 0; e < 16; ++e) A[e / RL + (e % RL) * (16 / RL)] = v[e];
    load_row(v, rowB);
    lds_barrier();
    block_fft<float, N1, -1, false, 0>(v, sre, sim, fresh_lane(t), tw());
    lds_barrier();
    store_lds(v);
    lds_barrier();
    {
      const int tl = fresh_lane(t);
      // the pair's global inputs (tables, PSD values) are fetched one
      // iteration ahead to overlap their latency
      auto fetch = [&](int j) {
        const int c = tl + NT * j;
        const int cm = N1 - 1 - c;
        const int k = rA + N2 * c, km = NC - k;
        const int64_t pa = int64_t(rA) * N1 + c, pb = int64_t(rB) * N1 + cm;
        return k < km ? long_pair_fetch<SRC>(a, psd, k, pa, pb) : long_pair_fetch<SRC>(a, psd, km, pb, pa);
      };
      LongPairIn nxt = fetch(0);
      // A stays in registers: each round of kTurn pairs works on the first
      // kTurn elements and moves them to the end
      constexpr int kTurn = 2;
#pragma unroll 1
      for (int j0 = 0; j0 < 16; j0 += kTurn) {
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
          const int j = j0 + u;
          const LongPairIn cur = nxt;
          nxt = fetch(min(j + 1, 15));
          const int c = tl + NT * j;
          const int cm = N1 - 1 - c;
          const int k = rA + N2 * c, km = NC - k;
          const int im = lpad<float>(cm);
          cpx<float> P = A[u], Q = {sre[im], sim[im]};
          if (k < km) long_pair<TP, SRC>(a, wsh, pr, cur, k, P, Q, flag);
          else long_pair<TP, SRC>(a, wsh, pr, cur, km, Q, P, flag);
          A[u] = P;
          sre[im] = Q.x;
          sim[im] = Q.y;
        }
        cpx<float> done[kTurn];
#pragma unroll
        for (int u = 0; u < kTurn; ++u) done[u] = A[u];
#pragma unroll
        for (int i = 0; i + kTurn < 16; ++i) A[i] = A[i + kTurn];
#pragma unroll
        for (int u = 0; u < kTurn; ++u) A[16 - kTurn + u] = done[u];
      }
    }
    lds_barrier();
    block_fft<float, N1, +1, true, 0>(v, sre, sim, fresh_lane(t), tw());
    store_row(v, rowB);
#pragma unroll
    for (int j = 0; j < 16; ++j) v[fft_in_slot<N1, 0>(j)] = A[j];
    lds_barrier();
    block_fft<float, N1, +1, false, 0>(v, sre, sim, fresh_lane(t), tw());
    store_row(v, rowA);
  }
  if (flag) atomicOr(&sflag, flag);
  __syncthreads();
  if (t == 0 && sflag && a.w.status) atomicOr(a.w.status + b, sflag);
}

template <int N1, int SRC>
void launch_cols_fwd(const LongArgs& a, int64_t items, hipStream_t st) {
  const dim3 grid(unsigned(N1 / 256), unsigned(items));
  if constexpr (N1 == 16384) {  // only N = 2^20 uses rows of 16384
    hipLaunchKernelGGL((k_long_cols_fwd<N1, 32, SRC>), grid, dim3(256), 0, st, a);
  } else {
    switch (a.N2) {
      case 4: hipLaunchKernelGGL((k_long_cols_fwd<N1, 4, SRC>), grid, dim3(256), 0, st, a); break;
      case 8: hipLaunchKernelGGL((k_long_cols_fwd<N1, 8, SRC>), grid, dim3(256), 0, st, a); break;
      case 16: hipLaunchKernelGGL((k_long_cols_fwd<N1, 16, SRC>), grid, dim3(256), 0, st, a); break;
      default: hipLaunchKernelGGL((k_long_cols_fwd<N1, 32, SRC>), grid, dim3(256), 0, st, a); break;
    }
  }
}

template <int N1, int SRC>
void launch_cols_inv(const LongArgs& a, int64_t items, hipStream_t st) {
  const dim3 grid(unsigned(N1 / 256), unsigned(items));
  if constexpr (N1 == 16384) {  // only N = 2^20 uses rows of 16384
    hipLaunchKernelGGL((k_long_cols_inv<N1, 32, SRC>), grid, dim3(256), 0, st, a);
  } else {
    switch (a.N2) {
      case 4: hipLaunchKernelGGL((k_long_cols_inv<N1, 4, SRC>), grid, dim3(256), 0, st, a); break;
      case 8: hipLaunchKernelGGL((k_long_cols_inv<N1, 8, SRC>), grid, dim3(256), 0, st, a); break;
      case 16: hipLaunchKernelGGL((k_long_cols_inv<N1, 16, SRC>), grid, dim3(256), 0, st, a); break;
      default: hipLaunchKernelGGL((k_long_cols_inv<N1, 32, SRC>), grid, dim3(256), 0, st, a); break;
    }
  }
}

// The passes of one window stage at row length N1 (see long_window).
template <int N1>
void long_passes(const DevCfg& d, int src, const LongArgs& a, const float* hdet, int64_t items, hipStream_t st) {
  const dim3 bins_grid(unsigned(N1 / 512), unsigned(items), unsigned(a.N2 / 2 + 1));
  const dim3 inject_grid(unsigned((a.NC / 2 + 1 + 255) / 256), unsigned(items));
  const dim3 rows_grid(unsigned(items * a.N2));
  if (src == 2) {
    hipLaunchKernelGGL((k_long_inject<N1>), inject_grid, dim3(256), 0, st, a, hdet);
    hipLaunchKernelGGL((k_long_rows<N1, +1>), rows_grid, dim3(N1 / 16), 0, st, a);
    launch_cols_inv<N1, 2>(a, items, st);
    return;
  }
  if (src == 0) launch_cols_fwd<N1, 0>(a, items, st);
  else launch_cols_fwd<N1, 1>(a, items, st);
  if (d.ord_win) {
    // rows, bins and inverse rows fused per row pair
    const dim3 pair_grid(unsigned(items * (a.N2 / 2)));
    if (src == 0) hipLaunchKernelGGL((k_long_rowpair<N1, double, 0>), pair_grid, dim3(N1 / 16), 0, st, a);
    else if (d.precision == 0) hipLaunchKernelGGL((k_long_rowpair<N1, float, 1>), pair_grid, dim3(N1 / 16), 0, st, a);
    else hipLaunchKernelGGL((k_long_rowpair<N1, double, 1>), pair_grid, dim3(N1 / 16), 0, st, a);
    launch_cols_inv<N1, 0>(a, items, st);
    return;
  }
  hipLaunchKernelGGL((k_long_rows<N1, -1>), rows_grid, dim3(N1 / 16), 0, st, a);
  if (src == 0) {
    hipLaunchKernelGGL((k_long_bins<N1, double, 0>), bins_grid, dim3(256), 0, st, a);
  } else if (d.precision == 0) {
    hipLaunchKernelGGL((k_long_bins<N1, float, 1>), bins_grid, dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL((k_long_bins<N1, double, 1>), bins_grid, dim3(256), 0, st, a);
  }
  hipLaunchKernelGGL((k_long_rows<N1, +1>), rows_grid, dim3(N1 / 16), 0, st, a);
  launch_cols_inv<N1, 0>(a, items, st);
}

}  // namespace

namespace gw {

int long_row_length(int NC) { return NC / 8192 <= 32 ? 8192 : 16384; }

// The window stage for N > 32768: SRC 0 whitens strain rows x, SRC 1 is the
// fused batch (x = background), SRC 2 injects hdet into the background
// noise.  w.out is [items][N] and doubles as the transform buffer.
gw_status long_window(gw_ctx* c, int src, const WinArgs& w, const float* x, const float* hdet, int64_t items,
                      hipStream_t st) {
  const DevCfg& d = c->dc;
  LongArgs a;
  a.w = w;
  a.twc = c->tw_long;
  a.twr = c->twr_win;
  a.tw1 = c->tw_win;
  a.x = x;
  a.NC = d.N / 2;
  const int N1 = long_row_length(a.NC);
  a.N2 = a.NC / N1;
  a.l2n2 = 0;
  while ((1 << a.l2n2) < a.N2) ++a.l2n2;
  const char* tabs = static_cast<const char*>(c->long_tabs);
  a.bins_t = reinterpret_cast<const BinTab*>(tabs);
  a.twr_t = reinterpret_cast<const cpx<float>*>(tabs + sizeof(BinTab) * size_t(a.NC));
  if (items <= 0) return GW_OK;
  if (items > 65535) return ctx_fail(c, GW_EINVAL, "long windows: at most 65535 (sample, detector) items per call");
  if (!c->long_tabs) return ctx_fail(c, GW_EUNSUPPORTED, "long windows need the binary32 tables");
  if (a.N2 < 4 || a.N2 > 32 || a.N2 * N1 != a.NC) return ctx_fail(c, GW_EUNSUPPORTED, "long windows: bad split");
  if (N1 == 8192) long_passes<8192>(d, src, a, hdet, items, st);
  else long_passes<16384>(d, src, a, hdet, items, st);
  return ctx_check_launch(c, src == 2 ? "long inject" : "long window");
}

}  // namespace gw
