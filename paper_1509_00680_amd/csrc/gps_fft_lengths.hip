// Two-level FFT passes for the lengths beside those of gps_fft_fast.hip: every
// even length of 16 to 448 and every odd one of 15 to 225 without a prime
// factor above 7 (the extents 15 to 225 and their doubles).  Longer and
// shorter lengths take the generic passes.
//
// The factor L1 of an even length is even, so that the zero half of a padded
// pencil is a compile-time half of each column; otherwise the two factors are
// as near to each other as the codelets allow, because a work-group holds B
// max(L1, L2) threads of which a transform step keeps B L2 or B L1 busy.
//
// These passes are bound as those of the tuned lengths are (latency of a tile's
// exchanges times the tiles in flight; memory on large grids).  Against the
// generic kernels, which sweep LDS once per radix with a barrier, an integer
// division and twiddles from global memory in each sweep, on one MI355X: vacuum
// solve of 100^3 (L = 200, mixed) 141.4 -> 64.0 us, of 28^3 to 60^3 1.35 to
// 1.4 x, generalized Poisson of 75 x 84 x 90 (L = 150, 168, 180, FP64) 13.36 ->
// 5.14 ms, other grids 1.5 to 2.5 x.
//
// Compiled once per group (GPS_LENGTH_GROUP), each group an object of its own,
// loaded by the first launch of one of its lengths.
#include "gps_fft_two.h"

#ifndef GPS_LENGTH_GROUP
#define GPS_LENGTH_GROUP 0
#endif

namespace gps {

// Row pairs per x-pass work-group: of 5 to 10, the count whose P max(L1, L2)
// threads waste the smallest share of their last wavefront (6 if several do).
constexpr int even_pairs(int m) {
  int best = 6;
  for (int P = 5; P <= 10; ++P)
    if (P * m * round64(best * m) > best * m * round64(P * m)) best = P;
  return best;
}

template <int A, int B, int P> static bool add_length() {
  bool ok = add_length_passes(TwoLevel<A, B, P, false>::passes());
  if constexpr (A * B <= kFewRowsLen)
    ok = add_few_rows_passes(TwoLevel<A, B, kFewRowsPairs, false>::x_passes32()) && ok;
  return ok;
}

#define GPS_LENGTH(A, B)           \
  static const bool len_##A##_##B = \
      add_length<A, B, even_pairs(larger(A, B))>();

#if GPS_LENGTH_GROUP == 0
GPS_LENGTH(4, 5)
GPS_LENGTH(8, 7)
GPS_LENGTH(9, 9)
GPS_LENGTH(14, 8)
GPS_LENGTH(12, 12)
GPS_LENGTH(18, 12)
GPS_LENGTH(28, 16)
#elif GPS_LENGTH_GROUP == 1
GPS_LENGTH(4, 7)
GPS_LENGTH(8, 5)
GPS_LENGTH(9, 7)
GPS_LENGTH(10, 10)
GPS_LENGTH(18, 9)
GPS_LENGTH(16, 15)
GPS_LENGTH(28, 14)
#elif GPS_LENGTH_GROUP == 2
GPS_LENGTH(9, 5)
GPS_LENGTH(10, 6)
GPS_LENGTH(10, 8)
GPS_LENGTH(15, 9)
GPS_LENGTH(20, 10)
GPS_LENGTH(14, 15)
GPS_LENGTH(24, 18)
#elif GPS_LENGTH_GROUP == 3
GPS_LENGTH(6, 4)
GPS_LENGTH(7, 7)
GPS_LENGTH(10, 5)
GPS_LENGTH(12, 7)
GPS_LENGTH(12, 15)
GPS_LENGTH(18, 14)
GPS_LENGTH(20, 21)
#elif GPS_LENGTH_GROUP == 4
GPS_LENGTH(9, 3)
GPS_LENGTH(6, 5)
GPS_LENGTH(6, 7)
GPS_LENGTH(14, 7)
GPS_LENGTH(16, 10)
GPS_LENGTH(18, 15)
GPS_LENGTH(20, 20)
#elif GPS_LENGTH_GROUP == 5
GPS_LENGTH(7, 5)
GPS_LENGTH(12, 9)
GPS_LENGTH(21, 7)
GPS_LENGTH(14, 12)
GPS_LENGTH(25, 7)
GPS_LENGTH(20, 14)
GPS_LENGTH(14, 25)
#elif GPS_LENGTH_GROUP == 6
GPS_LENGTH(5, 3)
GPS_LENGTH(7, 3)
GPS_LENGTH(6, 6)
GPS_LENGTH(12, 10)
GPS_LENGTH(10, 15)
GPS_LENGTH(21, 9)
GPS_LENGTH(18, 16)
GPS_LENGTH(18, 21)
#elif GPS_LENGTH_GROUP == 7
GPS_LENGTH(5, 5)
GPS_LENGTH(25, 5)
GPS_LENGTH(14, 9)
GPS_LENGTH(14, 10)
GPS_LENGTH(15, 15)
GPS_LENGTH(20, 15)
GPS_LENGTH(20, 18)
#elif GPS_LENGTH_GROUP == 8
GPS_LENGTH(6, 3)
GPS_LENGTH(6, 9)
GPS_LENGTH(10, 9)
GPS_LENGTH(15, 7)
GPS_LENGTH(14, 14)
GPS_LENGTH(14, 21)
GPS_LENGTH(16, 21)
#elif GPS_LENGTH_GROUP == 9
GPS_LENGTH(4, 4)
GPS_LENGTH(10, 7)
GPS_LENGTH(8, 9)
GPS_LENGTH(15, 5)
GPS_LENGTH(16, 14)
GPS_LENGTH(10, 25)
GPS_LENGTH(18, 18)
#endif
#undef GPS_LENGTH

}  // namespace gps
