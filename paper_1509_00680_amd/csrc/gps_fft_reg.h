// In-register FFT codelets with compile-time length (used by the two-level
// FFT passes).  Roots of unity are compile-time constants evaluated by the
// C++ front end in binary64 (Taylor series on the first octant), so the
// unrolled butterflies carry literal twiddles.
#pragma once

#include "gps_device.h"

namespace gps {

// ---- constexpr cos/sin(2 pi m / n) ------------------------------------------
// Evaluated in double-double arithmetic (Dekker's split product, Knuth's sum)
// and rounded once: the plain binary64 series is off by up to 2.3 units in the
// last place at N = 25.
struct DD {
  double hi, lo;
};
constexpr DD dd_sum(double a, double b) {            // a + b exactly
  const double s = a + b, t = s - a;
  return DD{s, (a - (s - t)) + (b - t)};
}
constexpr DD dd_prod(double a, double b) {           // a b exactly
  const double p = a * b;
  const double ca = 134217729.0 * a, ah = ca - (ca - a), al = a - ah;
  const double cb = 134217729.0 * b, bh = cb - (cb - b), bl = b - bh;
  return DD{p, ((ah * bh - p) + ah * bl + al * bh) + al * bl};
}
constexpr DD dd_add(DD a, DD b) {
  const DD s = dd_sum(a.hi, b.hi);
  return dd_sum(s.hi, s.lo + (a.lo + b.lo));
}
constexpr DD dd_mul(DD a, DD b) {
  const DD p = dd_prod(a.hi, b.hi);
  return dd_sum(p.hi, p.lo + (a.hi * b.lo + a.lo * b.hi));
}
constexpr DD dd_div(DD a, double b) {
  const double q = a.hi / b;
  const DD p = dd_prod(q, b);
  return dd_sum(q, (((a.hi - p.hi) - p.lo) + a.lo) / b);
}
// sum_i (-1)^i x^(2i+k) / (2i+k)!: sin (k = 1) and cos (k = 0) of 0 <= x <= pi/4
__host__ __device__ constexpr double ce_series(DD x, int k) {
  const DD x2 = dd_mul(x, x);
  DD term = k ? x : DD{1.0, 0.0}, sum = term;
  for (int i = 1; i < 14; ++i) {
    term = dd_div(dd_mul(term, x2), -(2.0 * i + k - 1.0) * (2.0 * i + k));
    sum = dd_add(sum, term);
  }
  return sum.hi;
}
// angle 2 pi m/n reduced to the first octant by exact integer symmetries
__host__ __device__ constexpr void ce_root(long long m, long long n, double* c, double* s) {
  m %= n;
  if (m < 0) m += n;
  // quadrant: multiply by 4 to compare with n exactly
  long long q = (4 * m) / n;            // 0..3
  long long r4 = 4 * m - q * n;         // angle within the quadrant, in units of 2 pi/(4n)
  // theta = 2 pi m/n = q pi/2 + phi, phi = (pi/2) r4/n
  bool swap = 2 * r4 > n;               // phi > pi/4: use pi/2 - phi
  long long num = swap ? (n - r4) : r4;
  const DD half_pi{1.5707963267948966, 6.123233995736766e-17};
  const DD phi = dd_div(dd_mul(half_pi, DD{(double)num, 0.0}), (double)n);
  double sp = ce_series(phi, 1), cp = ce_series(phi, 0);
  if (swap) { double t = sp; sp = cp; cp = t; }
  double cc = cp, ss = sp;
  if (q == 1) { cc = -sp; ss = cp; }
  else if (q == 2) { cc = -cp; ss = -sp; }
  else if (q == 3) { cc = sp; ss = -cp; }
  *c = cc;
  *s = ss;
}

// cos and sin(2 pi m / N), m < N, evaluated by the front end.
// KEPT: N = 8 and 16 with sqrt(1/2) and sin(pi/8) one unit in the last place below
// the nearest double, as a binary64 series gave them first.  An FP64 PCG solve
// multiplies a change of rounding by up to 1e8 before it reaches 1e-6 (solutions of
// 32^3 to 64^3 differ by 1e-8), so the common lengths round as they always did.
template <int N, bool KEPT> struct RootTable {
  double c[N], s[N];
  static constexpr double kept(double v) {
    constexpr double r[2] = {0.70710678118654757, 0.38268343236508978};
    constexpr double k[2] = {0.70710678118654746, 0.38268343236508973};
    for (int i = 0; i < 2; ++i) {
      if (v == r[i]) return k[i];
      if (v == -r[i]) return -k[i];
    }
    return v;
  }
  constexpr RootTable() : c{}, s{} {
    for (int m = 0; m < N; ++m) {
      ce_root(m, N, &c[m], &s[m]);
      if (KEPT && (N == 8 || N == 16)) {
        c[m] = kept(c[m]);
        s[m] = kept(s[m]);
      }
    }
  }
};
template <int N, bool KEPT> struct Roots2Pi { static constexpr RootTable<N, KEPT> t{}; };

// w_N^e = exp(-2 pi i e/N) (forward) or its conjugate (inverse), 0 <= e < N.
// Called with indices that are constant after unrolling, so the table reads
// fold to literals.
template <typename T, int N, bool INV, bool KEPT>
__device__ __forceinline__ cplx<T> croot(int e) {
  const double c = Roots2Pi<N, KEPT>::t.c[e], s = Roots2Pi<N, KEPT>::t.s[e];
  return cmk(T(c), T(INV ? s : -s));
}

// v * w_N^e for an exponent that is constant after unrolling: the quarter
// turns (1, -1, -i, +i) become swaps and sign changes instead of a full
// complex multiplication (whose products with 0 the compiler must keep).
template <typename T, int N, bool INV, bool KEPT>
__device__ __forceinline__ cplx<T> twiddle(cplx<T> v, int e) {
  e %= N;
  if (e == 0) return v;
  if (2 * e == N) return cmk(-v.x, -v.y);
  const bool minus_i = (4 * e == N) != INV;         // w = -i (else +i) when a quarter turn
  if (4 * e == N || 4 * e == 3 * N) return minus_i ? cmk(v.y, -v.x) : cmk(-v.y, v.x);
  return cmul(v, croot<T, N, INV, KEPT>(e));
}

// ---- small DFTs (radix butterflies) ---------------------------------------
template <int R> struct OddRoots;
template <> struct OddRoots<3> {
  static constexpr double c[2] = {1.0, -0.5};
  static constexpr double s[2] = {0.0, 0.86602540378443864676};
};
template <> struct OddRoots<5> {
  static constexpr double c[3] = {1.0, 0.30901699437494742410, -0.80901699437494742410};
  static constexpr double s[3] = {0.0, 0.95105651629515357212, 0.58778525229247312917};
};

template <> struct OddRoots<7> {
  static constexpr double c[4] = {1.0, 0.62348980185873353053, -0.22252093395631440429,
                                  -0.90096886790241912624};
  static constexpr double s[4] = {0.0, 0.78183148246802980871, 0.97492791218182360702,
                                  0.43388373911755812048};
};

template <typename T, bool INV, int R>
__device__ __forceinline__ void rdft(cplx<T>* x) {
  if constexpr (R == 2) {
    const cplx<T> a = x[0];
    x[0] = cadd(a, x[1]);
    x[1] = csub(a, x[1]);
  } else if constexpr (R == 4) {
    const cplx<T> a0 = cadd(x[0], x[2]), a1 = csub(x[0], x[2]);
    const cplx<T> a2 = cadd(x[1], x[3]), a3 = csub(x[1], x[3]);
    const cplx<T> ja3 = INV ? cmk(-a3.y, a3.x) : cmk(a3.y, -a3.x);
    x[0] = cadd(a0, a2);
    x[2] = csub(a0, a2);
    x[1] = cadd(a1, ja3);
    x[3] = csub(a1, ja3);
  } else {
    static_assert(R == 3 || R == 5 || R == 7, "radix");
    constexpr int H = (R - 1) / 2;
    cplx<T> a[H + 1], b[H + 1];
#pragma unroll
    for (int n = 1; n <= H; ++n) {
      a[n] = cadd(x[n], x[R - n]);
      b[n] = csub(x[n], x[R - n]);
    }
    const cplx<T> x0 = x[0];
    cplx<T> y0 = x0;
#pragma unroll
    for (int n = 1; n <= H; ++n) y0 = cadd(y0, a[n]);
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      cplx<T> re = x0, im = cmk(T(0), T(0));
#pragma unroll
      for (int n = 1; n <= H; ++n) {
        const int m = (n * k) % R;
        const int mf = m <= H ? m : R - m;
        re = cadd(re, cscale(a[n], T(OddRoots<R>::c[mf])));
        im = cadd(im, cscale(b[n], T(m <= H ? OddRoots<R>::s[mf] : -OddRoots<R>::s[mf])));
      }
      const cplx<T> mi = cmk(im.y, -im.x);   // -i * im
      if (INV) {
        x[k] = csub(re, mi);
        x[R - k] = cadd(re, mi);
      } else {
        x[k] = cadd(re, mi);
        x[R - k] = csub(re, mi);
      }
    }
    x[0] = y0;
  }
}

// ---- register Stockham over a compile-time radix list -----------------------
template <typename T, bool INV, bool KEPT, int N, int Ns, int... Rs> struct RegFFT {
  static __device__ __forceinline__ void run(cplx<T>*) {}
};
template <typename T, bool INV, bool KEPT, int N, int Ns, int R, int... Rest>
struct RegFFT<T, INV, KEPT, N, Ns, R, Rest...> {
  static __device__ __forceinline__ void run(cplx<T>* x) {
    cplx<T> y[N];
#pragma unroll
    for (int j = 0; j < N / R; ++j) {
      const int k = j % Ns;
      cplx<T> v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v[r] = x[j + r * (N / R)];
        if (r > 0 && k > 0) v[r] = twiddle<T, Ns * R, INV, KEPT>(v[r], r * k);
      }
      rdft<T, INV, R>(v);
      const int base = (j / Ns) * Ns * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) y[base + r * Ns] = v[r];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = y[i];
    RegFFT<T, INV, KEPT, N, Ns * R, Rest...>::run(x);
  }
};

// ---- prime-factor (Good-Thomas) codelet for N = N1 N2 with gcd(N1, N2) = 1 --
// Input n = (N2 n1 + N1 n2) mod N is read as a N1 x N2 array; N1-point DFTs
// along n1, then N2-point DFTs along n2, and output (k1, k2) is X[k] with
// k = k1 mod N1 = k2 mod N2 (Chinese remainder theorem).  The exponent of
// w_N factors exactly into w_N1^(n1 k1) w_N2^(n2 k2), so no twiddle factor
// sits between the two stages.  All indices are compile-time after unrolling.
// Inverse of a modulo m (gcd(a, m) = 1), evaluated in constant expressions.
__host__ __device__ constexpr int ce_modinv(int a, int m) {
  int r = 1;
  while ((a * r) % m != 1 % m) ++r;
  return r;
}
// CRT idempotents: E1 = 1 mod N1, 0 mod N2; E2 = 0 mod N1, 1 mod N2.  The
// output index of (k1, k2) is (k1 E1 + k2 E2) mod N, plain arithmetic on
// unrolled constants.
template <int N1, int N2> struct PfaMap {
  static constexpr int E1 = N2 * ce_modinv(N2 % N1, N1);
  static constexpr int E2 = N1 * ce_modinv(N1 % N2, N2);
};

template <typename T, bool INV, int N, bool KEPT> struct Codelet;

template <typename T, bool INV, int N1, int N2, bool KEPT> struct PfaFFT {
  static __device__ __forceinline__ void run(cplx<T>* x) {
    constexpr int N = N1 * N2;
    cplx<T> y[N];
#pragma unroll
    for (int n2 = 0; n2 < N2; ++n2) {
      cplx<T> v[N1];
#pragma unroll
      for (int n1 = 0; n1 < N1; ++n1) v[n1] = x[(N2 * n1 + N1 * n2) % N];
      Codelet<T, INV, N1, KEPT>::run(v);
#pragma unroll
      for (int k1 = 0; k1 < N1; ++k1) y[k1 * N2 + n2] = v[k1];
    }
#pragma unroll
    for (int k1 = 0; k1 < N1; ++k1) {
      cplx<T> v[N2];
#pragma unroll
      for (int n2 = 0; n2 < N2; ++n2) v[n2] = y[k1 * N2 + n2];
      Codelet<T, INV, N2, KEPT>::run(v);
#pragma unroll
      for (int k2 = 0; k2 < N2; ++k2)
        x[(k1 * PfaMap<N1, N2>::E1 + k2 * PfaMap<N1, N2>::E2) % N] = v[k2];
    }
  }
};

// Radix lists of the codelet lengths (prime-factor form where N splits into
// coprime factors).
#define GPS_CODELET(N, ...)                                                         \
  template <typename T, bool INV, bool KEPT> struct Codelet<T, INV, N, KEPT> {      \
    static __device__ __forceinline__ void run(cplx<T>* x) {                        \
      RegFFT<T, INV, KEPT, N, 1, __VA_ARGS__>::run(x);                              \
    }                                                                               \
  };
#define GPS_PFA_CODELET(N, N1, N2)                                                  \
  template <typename T, bool INV, bool KEPT> struct Codelet<T, INV, N, KEPT> {      \
    static __device__ __forceinline__ void run(cplx<T>* x) {                        \
      PfaFFT<T, INV, N1, N2, KEPT>::run(x);                                         \
    }                                                                               \
  };
GPS_CODELET(2, 2)
GPS_CODELET(3, 3)
GPS_CODELET(4, 4)
GPS_CODELET(5, 5)
GPS_CODELET(7, 7)
GPS_CODELET(8, 4, 2)
GPS_CODELET(9, 3, 3)
GPS_CODELET(16, 4, 4)
GPS_CODELET(25, 5, 5)
GPS_PFA_CODELET(6, 2, 3)
GPS_PFA_CODELET(10, 2, 5)
GPS_PFA_CODELET(12, 4, 3)
GPS_PFA_CODELET(14, 2, 7)
GPS_PFA_CODELET(15, 3, 5)
GPS_PFA_CODELET(18, 2, 9)
GPS_PFA_CODELET(20, 4, 5)
GPS_PFA_CODELET(21, 3, 7)
GPS_PFA_CODELET(24, 8, 3)
GPS_PFA_CODELET(28, 4, 7)
#undef GPS_CODELET
#undef GPS_PFA_CODELET

// Natural-order DFT of N values held in registers.
template <typename T, bool INV, int N, bool KEPT = false>
__device__ __forceinline__ void reg_fft(cplx<T>* x) {
  Codelet<T, INV, N, KEPT>::run(x);
}

}  // namespace gps
