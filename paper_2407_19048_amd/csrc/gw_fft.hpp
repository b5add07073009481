// Block-level FFT for gfx950: one workgroup transforms NC complex points,
// each of NT = NC/16 threads holding 16 of them in registers.
//
// Structure: Stockham auto-sort radix-R passes (radix 16 first, then 16s,
// then one 2/4/8 pass when NC is not a power of 16).  Inside a thread a pass
// is a radix-2 decimation-in-time DFT whose butterflies carry the inter-pass
// twiddles (see dit_fft).  Data is exchanged between passes through LDS, in
// separate real/imaginary planes padded (see pad_at) so that each pass's
// reads and writes are free of bank conflicts.
//
// Register layout of a thread t:
//   before the first pass   v[r]     = x[t + NT*r]                (r < 16)
//   after the last pass     v[m*R+r] = X[t + NT*m + r*NC/R]       (R = last radix)
// A thread therefore reads and writes coalesced global memory at both ends,
// with no transpose.
#pragma once
#include <hip/hip_runtime.h>

#include "gw_physics.hpp"

namespace gw {

template <class T> struct cpx { T x, y; };

template <class T> __device__ __forceinline__ cpx<T> cadd(cpx<T> a, cpx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <class T> __device__ __forceinline__ cpx<T> csub(cpx<T> a, cpx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <class T> __device__ __forceinline__ cpx<T> cmul(cpx<T> a, cpx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <class T> __device__ __forceinline__ cpx<T> cconj(cpx<T> a) { return {a.x, -a.y}; }
template <class T> __device__ __forceinline__ cpx<T> cscale(cpx<T> a, T s) { return {a.x * s, a.y * s}; }
// multiply by DIR*i (DIR = -1: by -i, DIR = +1: by +i)
template <int DIR, class T> __device__ __forceinline__ cpx<T> mul_i(cpx<T> a) {
  if constexpr (DIR < 0) return {a.y, -a.x};
  else return {-a.y, a.x};
}
// a * w for DIR = -1, a * conj(w) for DIR = +1 (w is a forward twiddle)
template <int DIR, class T> __device__ __forceinline__ cpx<T> twmul(cpx<T> a, cpx<T> w) {
  if constexpr (DIR < 0) return {a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x};
  else return {a.x * w.x + a.y * w.y, a.y * w.x - a.x * w.y};
}

// Returns p unchanged, but the compiler can no longer prove two loads through
// it the same: table loads stay next to the transform that uses them instead
// of being shared with (and kept live across) other transforms of the same
// kernel or loop iterations.  p points to global memory and is laundered as a
// global pointer, so that loads through it remain global loads: through a
// generic pointer they would become flat loads, which also count against the
// LDS wait counter and make every LDS barrier wait for them.
template <class T>
__device__ __forceinline__ const T* opaque(const T* p) {
  typedef const __attribute__((address_space(1))) T* gptr;
  gptr g = (gptr)p;
  asm volatile("" : "+s"(g));
  return (const T*)g;
}

// p (uniform over the workgroup) unchanged, but addresses derived from it are
// not shared with (and kept live across) other phases of the kernel that use
// the same pointer.
template <class T>
__device__ __forceinline__ T* fresh(T* p) {
  typedef __attribute__((address_space(1))) T* gptr;
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  // readfirstlane works on (signed) int: widen its result as unsigned, or a
  // low word with the top bit set would sign-extend into the high word
  const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(u))));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(u >> 32))));
  const uint64_t s = uint64_t(lo) | (uint64_t(hi) << 32);
  gptr g = (gptr)reinterpret_cast<T*>(s);
  asm volatile("" : "+s"(g));
  return (T*)g;
}

// The lane index t, unchanged, as a value the compiler cannot prove equal to
// t elsewhere: index and LDS-address arithmetic of one phase is then not
// shared with (and kept live across) the other phases.
__device__ __forceinline__ int fresh_lane(int t) {
  asm volatile("" : "+v"(t));
  return t;
}

// Workgroup barrier for the LDS exchanges: waits only for this wave's LDS
// operations (lgkmcnt) before s_barrier.  __syncthreads() also waits for
// every outstanding global load, which would expose the latency of loads
// issued ahead of time (next segment, next pass's twiddles) at each pass.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// LDS padding.  LDS has 32 banks of 4 bytes and serves a wavefront access to
// binary32 words 32 lanes per cycle.  In a binary32 plane, index i is stored
// at i + C (i >> 5): a run of 32 consecutive indices (every read of a pass,
// every natural-order access) then covers 32 banks for any C, and C is chosen
// per exchange for the stores of the pass that writes it (FftPad).  binary64
// planes keep one pad element every 16.
// pad_at(base, off) is the padded index of base + off for the index splits
// used here, where (base mod 32) + (off mod 32) < 32, so that the padding of
// base and of the compile-time offset off add up.
template <class T, int C> __device__ __forceinline__ int pad_at(int base, int off) {
  if constexpr (sizeof(T) == 4) {
    return base + C * (base >> 5) + off + C * (off >> 5);
  } else {
    const int i = base + off;
    return i + (i >> 4);
  }
}
// natural-order layout (C = 1)
template <class T> __device__ __forceinline__ int lpad(int i) { return pad_at<T, 1>(i, 0); }
// padding never moves an index beyond NC + NC/16 (C <= 2 in every plan)
template <int NC> struct LdsSize { static constexpr int value = NC + NC / 16; };

// a * exp(DIR * 2 pi i m / 16), m a compile-time constant
template <int M, int DIR, class T> __device__ __forceinline__ cpx<T> w16(cpx<T> a) {
  constexpr int m = ((M % 16) + 16) % 16;
  constexpr T C1 = T(0.92387953251128675613), S1 = T(0.38268343236508977173);
  constexpr T R2 = T(0.70710678118654752440);
  if constexpr (m == 0) return a;
  else if constexpr (m == 4) return mul_i<DIR>(a);
  else if constexpr (m == 8) return {-a.x, -a.y};
  else if constexpr (m == 12) return mul_i<-DIR>(a);
  else if constexpr (m == 2 || m == 6 || m == 10 || m == 14) {
    // exp(DIR i pi m/8) = (cx + DIR i sy)/sqrt2 with cx, sy in {+1,-1}
    constexpr T cx = (m == 2 || m == 14) ? T(1) : T(-1);
    constexpr T sy = (m == 2 || m == 6) ? T(1) : T(-1);
    constexpr T s = T(DIR) * sy;
    return {(a.x * cx - a.y * s) * R2, (a.y * cx + a.x * s) * R2};
  } else {
    // angle = quad * pi/2 + phi, phi = (m & 3) * pi/8 with (m & 3) in {1, 3}
    constexpr int q = m & 3;
    constexpr T cphi = (q == 1) ? C1 : S1, sphi = (q == 1) ? S1 : C1;
    constexpr int quad = m >> 2;
    constexpr T c = quad == 0 ? cphi : quad == 1 ? -sphi : quad == 2 ? -cphi : sphi;
    constexpr T sn = quad == 0 ? sphi : quad == 1 ? cphi : quad == 2 ? -sphi : -cphi;
    constexpr T s = T(DIR) * sn;
    return {a.x * c - a.y * s, a.y * c + a.x * s};
  }
}

template <int DIR, class T> __device__ __forceinline__ void dft2(cpx<T>* a) {
  cpx<T> t0 = a[0];
  a[0] = cadd(t0, a[1]);
  a[1] = csub(t0, a[1]);
}

template <int DIR, class T> __device__ __forceinline__ void dft4(cpx<T>& a0, cpx<T>& a1, cpx<T>& a2, cpx<T>& a3) {
  cpx<T> t0 = cadd(a0, a2), t1 = csub(a0, a2), t2 = cadd(a1, a3), t3 = mul_i<DIR>(csub(a1, a3));
  a0 = cadd(t0, t2);
  a2 = csub(t0, t2);
  a1 = cadd(t1, t3);
  a3 = csub(t1, t3);
}
template <int DIR, class T> __device__ __forceinline__ void dft4(cpx<T>* a) { dft4<DIR>(a[0], a[1], a[2], a[3]); }

template <int DIR, class T> __device__ __forceinline__ void dft8(cpx<T>* a) {
  cpx<T> e0 = a[0], e1 = a[2], e2 = a[4], e3 = a[6];
  cpx<T> o0 = a[1], o1 = a[3], o2 = a[5], o3 = a[7];
  dft4<DIR>(e0, e1, e2, e3);
  dft4<DIR>(o0, o1, o2, o3);
  o1 = w16<2, DIR>(o1);
  o2 = w16<4, DIR>(o2);
  o3 = w16<6, DIR>(o3);
  a[0] = cadd(e0, o0); a[4] = csub(e0, o0);
  a[1] = cadd(e1, o1); a[5] = csub(e1, o1);
  a[2] = cadd(e2, o2); a[6] = csub(e2, o2);
  a[3] = cadd(e3, o3); a[7] = csub(e3, o3);
}

// 16-point DFT as 4 x 4: X[k1 + 4 k2] = sum_n2 W4^(n2 k2) W16^(n2 k1) DFT4_n1(a[4 n1 + n2])[k1]
template <int DIR, class T> __device__ __forceinline__ void dft16(cpx<T>* a) {
  dft4<DIR>(a[0], a[4], a[8], a[12]);
  dft4<DIR>(a[1], a[5], a[9], a[13]);
  dft4<DIR>(a[2], a[6], a[10], a[14]);
  dft4<DIR>(a[3], a[7], a[11], a[15]);
  // after this, a[n2 + 4 k1] holds Y_{n2}[k1]
  a[5] = w16<1, DIR>(a[5]);
  a[9] = w16<2, DIR>(a[9]);
  a[13] = w16<3, DIR>(a[13]);
  a[6] = w16<2, DIR>(a[6]);
  a[10] = w16<4, DIR>(a[10]);
  a[14] = w16<6, DIR>(a[14]);
  a[7] = w16<3, DIR>(a[7]);
  a[11] = w16<6, DIR>(a[11]);
  a[15] = w16<9, DIR>(a[15]);
  dft4<DIR>(a[0], a[1], a[2], a[3]);
  dft4<DIR>(a[4], a[5], a[6], a[7]);
  dft4<DIR>(a[8], a[9], a[10], a[11]);
  dft4<DIR>(a[12], a[13], a[14], a[15]);
  // now a[4 k1 + k2] holds X[k1 + 4 k2]: transpose the 4x4 index
  cpx<T> t;
  t = a[1]; a[1] = a[4]; a[4] = t;
  t = a[2]; a[2] = a[8]; a[8] = t;
  t = a[3]; a[3] = a[12]; a[12] = t;
  t = a[6]; a[6] = a[9]; a[9] = t;
  t = a[7]; a[7] = a[13]; a[13] = t;
  t = a[11]; a[11] = a[14]; a[14] = t;
}

// exp(-2 pi i q / 16) for q = 1, 2, 3 as (cosine, tangent)
template <class T> __host__ __device__ constexpr cpx<T> root16(int q) {
  return q == 1 ? cpx<T>{T(0.92387953251128675613), T(-0.41421356237309504880)}
       : q == 2 ? cpx<T>{T(0.70710678118654752440), T(-1)}
                : cpx<T>{T(0.38268343236508977173), T(-2.41421356237309504880)};
}

// Butterfly e, o -> e + w o, e - w o with w = c (1 + i t) given as {c, t}
// (DIR = +1: with its conjugate), ROT: w further multiplied by DIR i.  Six
// fused multiply-adds: u + i v = (1 + i t) o takes two, the two outputs four.
template <int DIR, bool ROT, class T>
__device__ __forceinline__ void bfly(cpx<T> e, cpx<T> o, cpx<T> w, cpx<T>& s, cpx<T>& d) {
  const T t = DIR < 0 ? w.y : -w.y;
  const T u = fma_t(-t, o.y, o.x), v = fma_t(t, o.x, o.y);
  if constexpr (!ROT) {
    s = {fma_t(w.x, u, e.x), fma_t(w.x, v, e.y)};
    d = {fma_t(-w.x, u, e.x), fma_t(-w.x, v, e.y)};
  } else {
    constexpr T sg = T(-DIR);
    s = {fma_t(sg * w.x, v, e.x), fma_t(-sg * w.x, u, e.y)};
    d = {fma_t(-sg * w.x, v, e.x), fma_t(sg * w.x, u, e.y)};
  }
}

// The same with w = {cosine, sine}: eight, and no pole at the quarter turn.
template <int DIR, class T>
__device__ __forceinline__ void bfly_sine(cpx<T> e, cpx<T> o, cpx<T> w, cpx<T>& s, cpx<T>& d) {
  const T sn = DIR < 0 ? w.y : -w.y;
  s = {fma_t(-sn, o.y, fma_t(w.x, o.x, e.x)), fma_t(sn, o.x, fma_t(w.x, o.y, e.y))};
  d = {fma_t(sn, o.y, fma_t(-w.x, o.x, e.x)), fma_t(-sn, o.x, fma_t(-w.x, o.y, e.y))};
}

// Stage of DFT length LEN of the radix-R DFT below: butterflies of the pairs
// (q, q + LEN/2) of every run of LEN elements.
template <int R, int LEN, int DIR, bool TW, bool SINE, class T>
__device__ __forceinline__ void dit_stage(cpx<T>* b, const cpx<T>* w) {
#pragma unroll
  for (int g = 0; g < R; g += LEN)
#pragma unroll
    for (int q = 0; q < LEN / 2; ++q) {
      const bool rot = LEN >= 4 && q >= LEN / 4;  // the twiddle of q - LEN/4 times DIR i
      const int qq = rot ? q - LEN / 4 : q;
      const cpx<T> e = b[g + q], o = b[g + q + LEN / 2];
      cpx<T>&s = b[g + q], &d = b[g + q + LEN / 2];
      if constexpr (TW && SINE && LEN == 2) {
        bfly_sine<DIR>(e, o, w[0], s, d);
      } else if constexpr (TW) {
        const cpx<T> ww = w[LEN == 2 ? 0 : LEN / 4 + qq];
        if (rot) bfly<DIR, true>(e, o, ww, s, d);
        else bfly<DIR, false>(e, o, ww, s, d);
      } else if (qq == 0) {
        const cpx<T> r = rot ? mul_i<DIR>(o) : o;
        s = cadd(e, r);
        d = csub(e, r);
      } else {
        const cpx<T> ww = root16<T>(qq * (16 / LEN));
        if (rot) bfly<DIR, true>(e, o, ww, s, d);
        else bfly<DIR, false>(e, o, ww, s, d);
      }
    }
}

template <int R> __host__ __device__ constexpr int bit_reverse(int i) {
  int r = 0;
  for (int b = 1; b < R; b <<= 1) r = 2 * r + ((i & b) ? 1 : 0);
  return r;
}

// X[q] = sum_r W^r a[r] exp(DIR 2 pi i q r / R), in place, natural order in and
// out; W = 1 (TW false) or the pass's twiddle.  Radix-2 decimation in time:
// the stage of length LEN needs the twiddles W^(R/LEN) exp(-2 pi i q / LEN),
// of which those with q >= LEN/4 are -i times the others, so that a radix-R
// pass has R/2 distinct ones: w[0] for LEN = 2, w[LEN/4 + q] above, each as
// {cosine, tangent} (SINE: w[0] as {cosine, sine}).  A radix-16 pass with its twiddles is 192 fused
// multiply-adds, against 60 for multiplying 15 inputs by their twiddles plus
// 160 for a 4 x 4 DFT, and keeps 8 twiddles instead of 15.  A butterfly output
// takes two roundings instead of three, and the twiddles are rounded as pairs
// (see tan_twiddle): 1.18e-7 of a spectrum's norm at 4096 points.
template <int R, int DIR, bool TW, bool SINE, class T> __device__ __forceinline__ void dit_fft(cpx<T>* a, const cpx<T>* w) {
  cpx<T> b[R];
#pragma unroll
  for (int i = 0; i < R; ++i) b[i] = a[bit_reverse<R>(i)];
  dit_stage<R, 2, DIR, TW, SINE>(b, w);
  if constexpr (R >= 4) dit_stage<R, 4, DIR, TW, SINE>(b, w);
  if constexpr (R >= 8) dit_stage<R, 8, DIR, TW, SINE>(b, w);
  if constexpr (R >= 16) dit_stage<R, 16, DIR, TW, SINE>(b, w);
#pragma unroll
  for (int i = 0; i < R; ++i) a[i] = b[i];
}

// Radix plan: NP16 radix-16 passes and, when NC is not a power of 16, one
// pass of radix RL.  ORD 0 runs the small pass last, ORD 1 first (the two
// orderings trade LDS access patterns; an autotuner picks one per size).
template <int NC> struct FftPlan {
  static constexpr int NP16 = (NC >= 65536) ? 4 : (NC >= 4096) ? 3 : (NC >= 256) ? 2 : 1;
  static constexpr int RL = NC / (NP16 == 4 ? 65536 : NP16 == 3 ? 4096 : NP16 == 2 ? 256 : 16);
  static constexpr int NPASS = NP16 + (RL > 1 ? 1 : 0);
  static constexpr int NT = NC / 16;
  static_assert(NC == 1024 || NC == 2048 || NC == 4096 || NC == 8192 || NC == 16384, "unsupported FFT size");
};

template <int NC, int PASS, int ORD = 0> struct PassInfo {
  using P = FftPlan<NC>;
  static constexpr bool SMALL_FIRST = (ORD == 1) && (P::RL > 1);
  static constexpr int R = SMALL_FIRST ? (PASS == 0 ? P::RL : 16) : ((PASS < P::NP16) ? 16 : P::RL);
  static constexpr int p16 = SMALL_FIRST ? (PASS == 0 ? 0 : PASS - 1) : PASS;
  static constexpr int NS = SMALL_FIRST ? (PASS == 0 ? 1 : P::RL * (p16 == 0 ? 1 : p16 == 1 ? 16 : 256))
                                        : ((PASS == 0) ? 1 : (PASS == 1) ? 16 : (PASS == 2) ? 256 : 4096);
};

template <int NC, int ORD> struct PlanEnds {
  static constexpr int RFIRST = PassInfo<NC, 0, ORD>::R;
  static constexpr int RLAST = PassInfo<NC, FftPlan<NC>::NPASS - 1, ORD>::R;
};

// Padding constant of the exchange written by pass PASS.  Its stores form,
// per run of 32 lanes, 32/NS groups of NS consecutive indices NS*R apart
// (NS < 32) or one run of 32 consecutive indices (NS >= 32); C = 32/R puts
// the groups on disjoint banks.  With NS = 1 the stores are R apart and C = 1
// spreads them.
template <int NC, int PASS, int ORD> struct FftPad {
  static constexpr int R = PassInfo<NC, PASS, ORD>::R, NS = PassInfo<NC, PASS, ORD>::NS;
  static constexpr int C = (NS == 1 || NS >= 32) ? 1 : 32 / R;
  static_assert(NS == 1 || NS >= 32 || NS * R >= 32, "groups must be 32 words apart");
  static_assert(C <= 2, "padding must fit in LdsSize");
};

// Register slot of input x[t + NT*j] (j < 16) before the first pass.
template <int NC, int ORD = 0> __host__ __device__ constexpr int fft_in_slot(int j) {
  constexpr int R0 = PlanEnds<NC, ORD>::RFIRST, NB = 16 / R0;
  return (j % NB) * R0 + j / NB;
}

// Output bin held in element e after the last pass.
template <int NC, int ORD = 0> __device__ __forceinline__ int fft_out_index(int t, int e) {
  constexpr int R = PlanEnds<NC, ORD>::RLAST, NT = FftPlan<NC>::NT;
  return t + NT * (e / R) + (e % R) * (NC / R);
}

// Pass twiddle tables of a plan, one block per pass after the first, in pass
// order: for k < NS, the R/2 twiddles of dit_fft for W = exp(-2 pi i k / (NS R)),
// stored [max(R/4, 1)][NS][min(R/2, 2)] so that a wavefront, whose lanes hold
// consecutive k, reads consecutive entries of 8 or 16 bytes.  (The table
// W^n in n order was gathered at strides of up to 8 entries instead.)
template <int NC, int PASS, int ORD> struct PassTw {
  static constexpr int R = PassInfo<NC, PASS, ORD>::R, NS = PassInfo<NC, PASS, ORD>::NS, NB = 16 / R;
  static constexpr int G = R >= 4 ? 2 : 1;      // twiddles per table entry
  static constexpr int NG = R / 2 / G;          // entries per butterfly
  static constexpr int size = R / 2 * NS;       // cpx of the block
};
template <int NC, int PASS, int ORD> __host__ __device__ constexpr int pass_tw_offset() {
  if constexpr (PASS <= 1) return 0;
  else return pass_tw_offset<NC, PASS - 1, ORD>() + PassTw<NC, PASS - 1, ORD>::size;
}
// cpx of the tables of one order; the table of order 1 follows that of order 0
template <int NC, int ORD> struct PlanTw {
  static constexpr int size = pass_tw_offset<NC, FftPlan<NC>::NPASS, ORD>();
  static constexpr int offset = ORD == 0 ? 0 : PlanTw<NC, 0>::size;
};

// Tables for other transforms than Welch's hold the twiddle of a pass's first
// stage as {cosine, sine} in binary32.  There the pole's tangent, 2^28, would
// bound the data at 2^100 (spectra of windows with samples of 1e28 overflowed);
// now the largest tangent, NC/6, does.  Welch's squares overflow far below
// that, and binary64 has the range.  Two multiply-adds more in each butterfly
// of that stage: 2048 samples with a run filter take 280 us, 275 without.
// (2 e - s as the second output has six and no pole either, but its error is
// that of the larger output: coloured noise came out 5 % less accurate.)
template <class T> constexpr bool kSineTable = sizeof(T) == 4;

// The 8 twiddles of a thread's 16/R butterflies in pass PASS.
template <class T, int NC, int ORD> struct PassTwiddle {
  static constexpr bool kLate = false, kSine = kSineTable<T>;
  const cpx<T>* __restrict__ tab;  // tables of both orders
  template <int PASS> struct Regs { cpx<T> w[8]; };
  template <int PASS> __device__ __forceinline__ Regs<PASS> load(int t) const {
    using P = PassTw<NC, PASS, ORD>;
    constexpr int NT = NC / 16;
    const cpx<T>* p = tab + PlanTw<NC, ORD>::offset + pass_tw_offset<NC, PASS, ORD>();
    Regs<PASS> q;
#pragma unroll
    for (int m = 0; m < P::NB; ++m) {
      const int k = (t + NT * m) & (P::NS - 1);
#pragma unroll
      for (int g = 0; g < P::NG; ++g) {
        struct alignas(sizeof(cpx<T>) * P::G) Entry { cpx<T> e[P::G]; };
        const Entry v = reinterpret_cast<const Entry*>(p)[g * P::NS + k];
#pragma unroll
        for (int i = 0; i < P::G; ++i) q.w[m * (P::R / 2) + g * P::G + i] = v.e[i];
      }
    }
    return q;
  }
};

// All passes' twiddles held in registers (many transforms per thread).  (Welch's,
// from a table without sines.)
template <class T, int NC, int ORD> struct HeldTwiddle {
  static constexpr bool kLate = false, kSine = false;
  using Src = PassTwiddle<T, NC, ORD>;
  typename Src::template Regs<1> w1;
  typename Src::template Regs<2> w2;
  typename Src::template Regs<FftPlan<NC>::NPASS == 4 ? 3 : 2> w3;
  __device__ __forceinline__ void init(const cpx<T>* tab, int t) {
    const Src s{tab};
    w1 = s.template load<1>(t);
    w2 = s.template load<2>(t);
    if constexpr (FftPlan<NC>::NPASS == 4) w3 = s.template load<3>(t);
  }
  template <int PASS> __device__ __forceinline__ const auto& load(int) const {
    if constexpr (PASS == 1) return w1;
    else if constexpr (PASS == 2) return w2;
    else return w3;
  }
};

// Each pass's twiddles requested only after the arithmetic of the pass ahead
// of it, when that pass's own are dead (see block_fft): a binary64 transform
// whose thread also holds sums has no registers for two passes' twiddles.
template <class T, int NC, int ORD> struct LateTwiddle {
  static constexpr bool kLate = true, kSine = false;
  const cpx<T>* tab;
  __device__ __forceinline__ void init(const cpx<T>* tab_, int) { tab = tab_; }
  template <int PASS> __device__ __forceinline__ auto load(int t) const {
    return PassTwiddle<T, NC, ORD>{opaque(tab)}.template load<PASS>(fresh_lane(t));
  }
};

// One Stockham pass.  READ: take input from LDS (else registers already hold
// it).  WRITE: scatter the output to LDS (else it stays in registers in the
// final layout).  A barrier separates this pass's LDS reads from its writes;
// the caller must ensure the LDS buffer is free before a pass that WRITEs
// without READing.  w: the pass's 8 twiddles (unused in pass 0).  after() is
// called between the pass's arithmetic and its writes.
struct Nothing { __device__ __forceinline__ void operator()() const {} };
template <class T, int NC, int PASS, int DIR, bool READ, bool WRITE, int ORD, bool SINE, class After = Nothing>
__device__ __forceinline__ void fft_pass(cpx<T>* v, T* sre, T* sim, int t, const cpx<T>* w, After after = {}) {
  constexpr int R = PassInfo<NC, PASS, ORD>::R, NS = PassInfo<NC, PASS, ORD>::NS;
  constexpr int NT = NC / 16, NB = 16 / R, STRIDE = NC / R;
  // layout of the buffer read: written by the previous pass, or natural order
  constexpr int CR = (PASS == 0) ? 1 : FftPad<NC, (PASS > 0 ? PASS - 1 : 0), ORD>::C;
  constexpr int CW = FftPad<NC, PASS, ORD>::C;
  if constexpr (READ) {
#pragma unroll
    for (int m = 0; m < NB; ++m) {
      const int j = t + NT * m;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int i = pad_at<T, CR>(j, r * STRIDE);
        v[m * R + r] = {sre[i], sim[i]};
      }
    }
  }
#pragma unroll
  for (int m = 0; m < NB; ++m) dit_fft<R, DIR, (NS > 1), SINE>(v + m * R, w + m * (R / 2));
  after();
  if constexpr (WRITE) {
    if constexpr (READ) lds_barrier();
#pragma unroll
    for (int m = 0; m < NB; ++m) {
      const int j = t + NT * m;
      const int k = j & (NS - 1);
      const int base = (j - k) * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int i = pad_at<T, CW>(base, r * NS);
        sre[i] = v[m * R + r].x;
        sim[i] = v[m * R + r].y;
      }
    }
    lds_barrier();
  }
}

// Whole transform.  FIRST_FROM_LDS: the first pass reads its input from LDS
// in natural order (else v holds it: x[t + NT j] in slot fft_in_slot(j)).
// The result stays in registers in the final layout (see fft_out_index).
// Ends with LDS still being read by other threads: barrier before reusing it.
// Each pass's twiddles are requested before the pass ahead of it, so that
// their latency is hidden behind that pass.  Late twiddles (three passes) are
// requested behind its arithmetic; ahead() is then called after the last
// request, for loads of the caller's that take longer: loads return in order.
template <class T, int NC, int DIR, bool FIRST_FROM_LDS, int ORD = 0, class TW, class Ahead = Nothing>
__device__ __forceinline__ void block_fft(cpx<T>* v, T* sre, T* sim, int t, const TW& tw, Ahead ahead = {}) {
  if constexpr (TW::kLate) {
    static_assert(FftPlan<NC>::NPASS == 3, "three passes");
    using Src = PassTwiddle<T, NC, ORD>;
    typename Src::template Regs<1> w1;
    typename Src::template Regs<2> w2;
    fft_pass<T, NC, 0, DIR, FIRST_FROM_LDS, true, ORD, TW::kSine>(v, sre, sim, t, nullptr,
                                                       [&]() { w1 = tw.template load<1>(t); });
    fft_pass<T, NC, 1, DIR, true, true, ORD, TW::kSine>(v, sre, sim, t, w1.w, [&]() {
      w2 = tw.template load<2>(t);
      ahead();
    });
    fft_pass<T, NC, 2, DIR, true, false, ORD, TW::kSine>(v, sre, sim, t, w2.w);
  } else {
    const auto w1 = tw.template load<1>(t);
    fft_pass<T, NC, 0, DIR, FIRST_FROM_LDS, true, ORD, TW::kSine>(v, sre, sim, t, w1.w);
    const auto w2 = tw.template load<2>(t);
    fft_pass<T, NC, 1, DIR, true, true, ORD, TW::kSine>(v, sre, sim, t, w1.w);
    if constexpr (FftPlan<NC>::NPASS == 3) {
      fft_pass<T, NC, 2, DIR, true, false, ORD, TW::kSine>(v, sre, sim, t, w2.w);
    } else {
      const auto w3 = tw.template load<3>(t);
      fft_pass<T, NC, 2, DIR, true, true, ORD, TW::kSine>(v, sre, sim, t, w2.w);
      fft_pass<T, NC, 3, DIR, true, false, ORD, TW::kSine>(v, sre, sim, t, w3.w);
    }
  }
}

}  // namespace gw
