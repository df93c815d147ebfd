// Two-level FFT passes: the table of lengths, and the lengths of the common
// grids (tuned tiles; gps_fft_lengths.hip holds the others).
#include "gps_fft_two.h"

namespace gps {

// Row pairs per work-group of the x passes: 6, and 10 at length 320 (L1 =
// 20).  Every x-forward work-group re-sums the x-inverse's partials, one per
// work-group, so that head costs the square of the work-group count; at
// 160^3 (12,800 row pairs) 10 pairs take the x forward from 39.1 to 32.2 us
// (8 and 12 pairs: 36.1 us); on the 96^3 and 128 x 128 x 192 grids 6 pairs
// are fastest.
template <int L1> constexpr int xpairs() { return L1 == 20 ? 10 : 6; }

// Zero-initialised before any entry adds itself.
static LengthPasses g_passes[kMaxFastLen + 1];

bool add_length_passes(const LengthPasses& e) {
  if (e.L < 1 || e.L > kMaxFastLen) return false;
  g_passes[e.L] = e;
  return true;
}

#define GPS_TUNED_LENGTH(A, B) \
  static const bool tuned_##A##_##B = add_length_passes(TwoLevel<A, B, xpairs<A>(), true>::passes());
GPS_TUNED_LENGTH(8, 4)
GPS_TUNED_LENGTH(8, 6)
GPS_TUNED_LENGTH(8, 8)
GPS_TUNED_LENGTH(12, 8)
GPS_TUNED_LENGTH(16, 8)
GPS_TUNED_LENGTH(16, 12)
GPS_TUNED_LENGTH(16, 16)
GPS_TUNED_LENGTH(20, 16)
GPS_TUNED_LENGTH(24, 16)
#undef GPS_TUNED_LENGTH

bool fast_length(int L) { return L >= 1 && L <= kMaxFastLen && g_passes[L].L == L; }

// Partials of the solve-mode x passes: one per work-group.
int fast_xpass_parts(int L, int nrows) {
  const int P = g_passes[L].P;
  return ((nrows + 1) / 2 + P - 1) / P;
}

// As the arrays of k_fxinv: KP pairs of rows from both parities, EOUT points with
// their five fields (six with the mean term), ETW twiddles, the shares of delta (and mu).
int fast_xinv_values(int L, int lout, int periodic_mean) {
  const LengthPasses& e = g_passes[L];
  const int NT = xthreads(e.L1, e.L2, e.P), KS = NT / e.P;
  const int KP = (L / 2 + 1 + KS - 1) / KS, EOUT = (2 * e.P * lout + NT - 1) / NT;
  const int shares = (NT == 64 ? 16 : 8) * (periodic_mean ? 2 : 1);
  return 8 * KP + (periodic_mean ? 6 : 5) * EOUT + 2 * ((L + NT - 1) / NT) + 2 * shares;
}

// z pass (solve mode): one partial per wavefront
template <typename T> int fast_strided_parts(const SParams<T>& p) {
  const LengthPasses& e = g_passes[p.L];
  const int B = strided_tile<T>(p.L), W = B * kStridedTiles;
  return (p.npencils + W - 1) / W * (round64(B * larger(e.L1, e.L2)) / 64);
}
template int fast_strided_parts<float>(const SParams<float>&);
template int fast_strided_parts<double>(const SParams<double>&);

template <> bool fast_strided<float>(int mode, const SParams<float>& p, hipStream_t s) {
  if (!fast_length(p.L)) return false;
  g_passes[p.L].strided32(mode, p, s);
  return true;
}
template <> bool fast_strided<double>(int mode, const SParams<double>& p, hipStream_t s) {
  if (!fast_length(p.L)) return false;
  g_passes[p.L].strided64(mode, p, s);
  return true;
}
template <> bool fast_xfwd<float>(int mode, const XParams<float>& p, hipStream_t s) {
  return fast_length(p.g.Lx) && g_passes[p.g.Lx].xfwd32(mode, p, s);
}
template <> bool fast_xfwd<double>(int mode, const XParams<double>& p, hipStream_t s) {
  return fast_length(p.g.Lx) && g_passes[p.g.Lx].xfwd64(mode, p, s);
}
template <> bool fast_xinv<float>(int mode, const XParams<float>& p, hipStream_t s) {
  return fast_length(p.g.Lx) && g_passes[p.g.Lx].xinv32(mode, p, s);
}
template <> bool fast_xinv<double>(int mode, const XParams<double>& p, hipStream_t s) {
  return fast_length(p.g.Lx) && g_passes[p.g.Lx].xinv64(mode, p, s);
}

}  // namespace gps
