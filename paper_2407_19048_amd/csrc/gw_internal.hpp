// Host-side definitions shared by the library's translation units.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <functional>
#include <string>
#include <vector>

#include "gw_fft.hpp"
#include "gw_physics.hpp"
#include "../../include/gwgen.h"

struct gw_ctx {
  gw_config cfg;
  gw::DevCfg dc;
  double* kcbrt = nullptr;    // [F]  k^(1/3)
  double* lnk3 = nullptr;     // [F]  ln(k)/3
  double* k53 = nullptr;      // [F]  k^(-5/3) (0 at k = 0)
  void* tw_win = nullptr;     // pass twiddle tables of the window (or row) transform, both orders
  void* twr_win = nullptr;    // cpx<T>[N/4 + 1]
  void* tw_welch = nullptr;   // Welch table of L (WelchTab)
  void* tw_long = nullptr;    // cpx<float>[N2][N1]: W_NC^(m1 k2), windows longer than 32768 samples
  // windows longer than 32768 samples: BinTab[N/2] and exp(-2 pi i k / N)
  // (cpx<float>[N/2]) for k < N/2, stored at the position (k mod N2) N1 + k / N2
  // of bin k in the transposed four-step spectrum
  void* long_tabs = nullptr;
  int device = 0;             // HIP device the context was created on
  int n_cu = 256;             // its compute units
  void* scratch = nullptr;    // that device's copy of the library's static scratch area
  std::string err;
};

// A captured batch pipeline; each launch advances the device batch counter.
struct gw_graph {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  uint64_t* batch = nullptr;  // device batch index inside the caller's workspace
  std::string err;
};

namespace gw {
// Autotuners time every variant once per round and keep each one's best round.
constexpr int kTuneRounds = 3;
struct WinArgs;
gw_status ctx_fail(gw_ctx* c, gw_status s, const std::string& msg);
// Window stage of windows longer than 32768 samples (four-step transforms
// in the output buffer): src 0 whiten, 1 fused batch, 2 inject.
gw_status long_window(gw_ctx* c, int src, const WinArgs& w, const float* x, const float* hdet, int64_t items,
                      hipStream_t st);
// Row length N1 of the four-step split NC = N1 x N2 of those windows.
int long_row_length(int NC);
gw_status ctx_check_launch(gw_ctx* c, const char* what);
// Host validation of a configuration into device constants (nothing launched).
gw_status validate_config(const gw_config* g, DevCfg* dc, std::string* why);
gw_status capture_graph(const std::function<gw_status(hipStream_t)>& enqueue, uint64_t* batch, uint64_t first,
                        gw_graph** out, std::string* why);

// Long windows' table entry of a bin: ln(k)/3 and k^(-5/3) (both 0 at k = 0).
struct alignas(16) BinTab { double lk = 0.0, k53 = 0.0; };

// {cosine, tangent} of the angle -2 pi num / den, 0 <= num <= den / 2.  In
// binary32 they are rounded as a pair, {c, t} with c (1 + i t) closest to the
// twiddle: t the rounded tangent or one of its neighbours, c the rounded best
// factor to it.  Rounded by themselves they left a twiddle's modulus up to
// twice the rounding error, which a PSD does not average over its segments:
// 7.3e-8 of a PSD's norm at 4096 points, 4.7e-8 so.
// At the quarter turn, where the tangent has no value, the cosine is set to
// 2^-28 (binary32) or 2^-56: a quarter of a unit in the last place of the sine,
// and still far from overflow when a value is multiplied by the tangent.
template <class T>
inline cpx<T> tan_twiddle(int64_t num, int64_t den) {
  if (4 * num == den) {
    const T tiny = sizeof(T) == 4 ? T(0x1p-28) : T(0x1p-56);
    return {tiny, T(-1) / tiny};
  }
  double sn, cs;
  ::sincos(-2.0 * M_PI * double(num) / double(den), &sn, &cs);
  const double tn = sn / cs;
  cpx<T> best = {T(cs), T(tn)};
  if constexpr (sizeof(T) == 4) {
    uint32_t bits;
    std::memcpy(&bits, &best.y, 4);
    double least = 4.0;
    for (const uint32_t b : {bits, bits - 1, bits + 1}) {  // (below 0 a NaN, which is no less)
      float t;
      std::memcpy(&t, &b, 4);
      // (cs + sn t) / (1 + t^2), to the first order in t - tn
      const float c = float(cs - cs * cs * sn * (t - tn));
      const double dx = c - cs, dy = double(c) * t - sn, e = dx * dx + dy * dy;
      if (e < least) {
        least = e;
        best = {c, t};
      }
    }
  }
  return best;
}

template <class T>
inline cpx<T> sin_twiddle(int64_t num, int64_t den) {
  const double ang = -2.0 * M_PI * double(num) / double(den);
  return {T(std::cos(ang)), T(std::sin(ang))};
}

template <class T, int NC, int ORD, int PASS>
inline void append_pass_table(std::vector<cpx<T>>& h, bool sine) {
  if constexpr (PASS < FftPlan<NC>::NPASS) {
    using P = PassTw<NC, PASS, ORD>;
    const size_t at = h.size();
    h.resize(at + P::size);
    for (int k = 0; k < P::NS; ++k)
      for (int len = 2; len <= P::R; len *= 2)
        for (int q = 0; q < (len >= 4 ? len / 4 : 1); ++q) {
          // W^(R/len) exp(-2 pi i q / len), W = exp(-2 pi i k / (NS R))
          const int i = len == 2 ? 0 : len / 4 + q;
          const int64_t num = int64_t(k) + int64_t(q) * P::NS, den = int64_t(P::NS) * len;
          h[at + (size_t(i / P::G) * P::NS + k) * P::G + i % P::G] =
              sine && len == 2 ? sin_twiddle<T>(num, den) : tan_twiddle<T>(num, den);
        }
    append_pass_table<T, NC, ORD, PASS + 1>(h, sine);
  }
}

// Pass twiddle tables of an nc-point transform (see PassTw), order 0 then 1;
// sine: the first stages' twiddles as sines (see kSineTable).
template <class T, int NC>
inline std::vector<cpx<T>> plan_tables_of(bool sine) {
  std::vector<cpx<T>> h;
  append_pass_table<T, NC, 0, 1>(h, sine);
  append_pass_table<T, NC, 1, 1>(h, sine);
  return h;
}
template <class T>
inline std::vector<cpx<T>> plan_tables(int nc, bool sine = kSineTable<T>) {
  switch (nc) {
    case 1024: return plan_tables_of<T, 1024>(sine);
    case 2048: return plan_tables_of<T, 2048>(sine);
    case 4096: return plan_tables_of<T, 4096>(sine);
    case 8192: return plan_tables_of<T, 8192>(sine);
    default: return plan_tables_of<T, 16384>(sine);
  }
}

// The Welch table of L = l (WelchTab): pass twiddles, the window's first half.
template <class T>
inline std::vector<cpx<T>> welch_tables(int l) {
  std::vector<cpx<T>> h = plan_tables<T>(l, false);
  auto hann = [&](int n) {
    const double sp = std::sin(M_PI * double(n) / double(l));
    return T(sp * sp);
  };
  for (int n = 0; n < l / 2; n += 2) h.push_back({hann(n), hann(n + 1)});
  return h;
}
}  // namespace gw
