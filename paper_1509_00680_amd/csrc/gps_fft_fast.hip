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
static LengthPasses g_few_rows[kFewRowsLen + 1];

bool add_length_passes(const LengthPasses& e) {
  if (e.L < 1 || e.L > kMaxFastLen) return false;
  g_passes[e.L] = e;
  return true;
}

bool add_few_rows_passes(const LengthPasses& e) {
  if (e.L < 1 || e.L > kFewRowsLen) return false;
  g_few_rows[e.L] = e;
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
// (After them: this order is the kernels' order in the code object, and an iteration
// of 96^3 takes three kernels that about fill the instruction cache.  With these
// between the others the same kernels lay elsewhere and the solve took 3.60 instead of
// 3.54 ms.)
#define GPS_FEW_ROWS(A, B)             \
  static const bool few_##A##_##B = \
      add_few_rows_passes(TwoLevel<A, B, kFewRowsPairs, true>::x_passes32());
GPS_FEW_ROWS(8, 4)
GPS_FEW_ROWS(8, 6)
GPS_FEW_ROWS(8, 8)
#undef GPS_FEW_ROWS

bool fast_length(int L) { return L >= 1 && L <= kMaxFastLen && g_passes[L].L == L; }

// FP32 x passes of every length up to 64 on grids of up to 4096 rows take four row
// pairs per work-group.  Such a grid is bound by the latency of a work-group, and six to
// ten pairs leave most CUs without one (32^3: 86 of 256).  Four pairs against the length's own
// count, solves and vacuum solves of 41 grids at 18 of the 24 lengths: vacuum 1.00 to 1.07 x (one at
// 0.995), solves 1.00 to 1.07 (two at 0.98), mean 1.025; 32^3 at 1e-6 1003 -> 958 us.  Longer
// lengths with four pairs on as few rows: 70 to 90, 108 and 120 1.01 to 1.05, but 96, 98, 100,
// 126 and 128 0.95 to 1.01.  More rows: 160 x 160 x 48 (25,600, of which 3200 work-groups each
// re-sum as many partials) 0.98.  FP32 only: the order of the partial sums is part of an
// FP64 solve's rounding, which PCG amplifies (Roots2Pi).
template <typename T> static const LengthPasses& x_passes(int L, int nrows) {
  if (sizeof(T) == sizeof(float) && L <= kFewRowsLen && nrows <= kFewRows) return g_few_rows[L];
  return g_passes[L];
}

template <typename T> bool fast_solve(const XParams<T>& p) {
  if (!fast_length(p.g.Lx)) return false;
  return sizeof(T) == sizeof(float) || g_passes[p.g.Lx].six64 || p.Lin != p.g.Lx ||
         !(p.refine || p.periodic_mean);
}
template bool fast_solve<float>(const XParams<float>&);
template bool fast_solve<double>(const XParams<double>&);

// Partials of the solve-mode x passes: one per work-group.
template <typename T> int fast_xpass_parts(int L, int nrows) {
  const int P = x_passes<T>(L, nrows).P;
  return ((nrows + 1) / 2 + P - 1) / P;
}
template int fast_xpass_parts<float>(int, int);
template int fast_xpass_parts<double>(int, int);

// As the arrays of k_fxinv: KP pairs of rows from both parities, EOUT points with
// their five fields (six with the mean term), ETW twiddles, the shares of delta (and mu).
// (g_passes: the rule that asks is for grids beyond the few rows.)
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
  return fast_length(p.g.Lx) && x_passes<float>(p.g.Lx, p.nrows).xfwd32(mode, p, s);
}
template <> bool fast_xfwd<double>(int mode, const XParams<double>& p, hipStream_t s) {
  return fast_length(p.g.Lx) && x_passes<double>(p.g.Lx, p.nrows).xfwd64(mode, p, s);
}
template <> bool fast_xinv<float>(int mode, const XParams<float>& p, hipStream_t s) {
  return fast_length(p.g.Lx) && x_passes<float>(p.g.Lx, p.nrows).xinv32(mode, p, s);
}
template <> bool fast_xinv<double>(int mode, const XParams<double>& p, hipStream_t s) {
  return fast_length(p.g.Lx) && x_passes<double>(p.g.Lx, p.nrows).xinv64(mode, p, s);
}

}  // namespace gps
