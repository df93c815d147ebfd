// FFT passes of the vacuum Poisson solver used as PCG preconditioner
// (Eq. PCGdef: v = S^-1 G S^-1 r, G a zero-padded FFT convolution).
//
// Every pass keeps one tile of pencils in LDS and runs a self-sorting
// (Stockham) mixed-radix FFT on it.  Tiles hold B adjacent pencils with the
// pencil index fastest, so global loads and stores of a tile row are
// contiguous.  Zero padding is pruned: the zero half of a padded axis is
// never read from or written to HBM.
//
//   x pass   two real rows packed as one complex row (R2C / C2R pairing);
//            fused prologue r/sqrt(eps) and epilogue u/sqrt(eps) + (v, r).
//   y pass   strided C2C, in place in the work buffer.
//   z pass   strided C2C forward, multiply by the real even Green's
//            spectrum, C2C inverse, all in one pass through LDS.
#include <algorithm>

#include "gps_fft_plane.h"
#include "gps_iter.h"
#include "gps_launch.h"
#include "gps_sc.h"

namespace gps {

// ---------------------------------------------------------------------------
// small DFTs
// ---------------------------------------------------------------------------
template <int R> struct Roots;
template <> struct Roots<3> {
  static constexpr double c[2] = {1.0, -0.5};
  static constexpr double s[2] = {0.0, 0.86602540378443864676};
};
template <> struct Roots<5> {
  static constexpr double c[3] = {1.0, 0.30901699437494742410, -0.80901699437494742410};
  static constexpr double s[3] = {0.0, 0.95105651629515357212, 0.58778525229247312917};
};
template <> struct Roots<7> {
  static constexpr double c[4] = {1.0, 0.62348980185873353053, -0.22252093395631440429,
                                  -0.90096886790241912624};
  static constexpr double s[4] = {0.0, 0.78183148246802980871, 0.97492791218182360702,
                                  0.43388373911755812048};
};

// y_k = sum_n x_n w^(nk), w = exp(-2 pi i/R) (forward) or its conjugate.
template <typename T, bool INV, int R>
__device__ __forceinline__ void dft(cplx<T>* x) {
  if constexpr (R == 2) {
    cplx<T> a = x[0];
    x[0] = cadd(a, x[1]);
    x[1] = csub(a, x[1]);
  } else if constexpr (R == 4) {
    cplx<T> a0 = cadd(x[0], x[2]), a1 = csub(x[0], x[2]);
    cplx<T> a2 = cadd(x[1], x[3]), a3 = csub(x[1], x[3]);
    // forward: (-i) a3 ; inverse: (+i) a3
    cplx<T> ja3 = INV ? cmk(-a3.y, a3.x) : cmk(a3.y, -a3.x);
    x[0] = cadd(a0, a2);
    x[2] = csub(a0, a2);
    x[1] = cadd(a1, ja3);
    x[3] = csub(a1, ja3);
  } else {
    constexpr int H = (R - 1) / 2;
    cplx<T> a[H + 1], b[H + 1];
#pragma unroll
    for (int n = 1; n <= H; ++n) {
      a[n] = cadd(x[n], x[R - n]);
      b[n] = csub(x[n], x[R - n]);
    }
    cplx<T> x0 = x[0];
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
        const T cs = T(Roots<R>::c[mf]);
        const T sn = T(m <= H ? Roots<R>::s[mf] : -Roots<R>::s[mf]);
        re = cadd(re, cscale(a[n], cs));
        im = cadd(im, cscale(b[n], sn));
      }
      // y_k = re - i im (forward), y_{R-k} = re + i im
      cplx<T> mi = cmk(im.y, -im.x);   // -i * im
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

// One Stockham stage of radix R over a tile of B = 2^lgB pencils of length L
// stored as buf[t * B + b].  Ns = product of the radices of earlier stages.
template <typename T, bool INV, int R>
__device__ __forceinline__ void stage(cplx<T>* __restrict__ buf, int L, int lgB, int Ns,
                                      const cplx<T>* __restrict__ tw) {
  constexpr int MAXE = TileCap<T>::elems;
  constexpr int MAXBF = (MAXE + R * kThreads - 1) / (R * kThreads);
  const int B = 1 << lgB;
  const int LR = L / R;
  const int nbf = LR << lgB;
  const int twstride = L / (Ns * R);
  const int tid = threadIdx.x;
  cplx<T> x[MAXBF][R];
#pragma unroll
  for (int i = 0; i < MAXBF; ++i) {
    const int e = tid + i * kThreads;
    if (e < nbf) {
      const int b = e & (B - 1);
      const int j = e >> lgB;
#pragma unroll
      for (int r = 0; r < R; ++r) x[i][r] = buf[((j + r * LR) << lgB) + b];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MAXBF; ++i) {
    const int e = tid + i * kThreads;
    if (e < nbf) {
      const int b = e & (B - 1);
      const int j = e >> lgB;
      const int jq = j / Ns;
      const int k = j - jq * Ns;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        cplx<T> w = tw[r * k * twstride];
        if (INV) w.y = -w.y;
        x[i][r] = cmul(x[i][r], w);
      }
      dft<T, INV, R>(x[i]);
      const int base = jq * Ns * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) buf[((base + r * Ns) << lgB) + b] = x[i][r];
    }
  }
  __syncthreads();
}

template <typename T, bool INV>
__device__ void lds_fft(cplx<T>* buf, int L, int lgB, const RadixPlan& rp,
                        const cplx<T>* __restrict__ tw) {
  int Ns = 1;
  for (int s = 0; s < rp.nstages; ++s) {
    const int R = rp.radix[s];
    switch (R) {
      case 4: stage<T, INV, 4>(buf, L, lgB, Ns, tw); break;
      case 2: stage<T, INV, 2>(buf, L, lgB, Ns, tw); break;
      case 3: stage<T, INV, 3>(buf, L, lgB, Ns, tw); break;
      case 5: stage<T, INV, 5>(buf, L, lgB, Ns, tw); break;
      default: stage<T, INV, 7>(buf, L, lgB, Ns, tw); break;
    }
    Ns *= R;
  }
}

// ---------------------------------------------------------------------------
// cell-averaged 1/r (free-boundary Green's function, plan time, FP64)
// ---------------------------------------------------------------------------
// F with d^3F/dxdydz = 1/|r| (x, y, z nonzero).
__device__ double prism_antiderivative(double x, double y, double z) {
  const double r = sqrt(x * x + y * y + z * z);
  return y * z * log(x + r) + x * z * log(y + r) + x * y * log(z + r)
         - 0.5 * x * x * atan(y * z / (x * r)) - 0.5 * y * y * atan(x * z / (y * r))
         - 0.5 * z * z * atan(x * y / (z * r));
}

// Integral of 1/|u| over the unit cube centred at (mx, my, mz), mx, my, mz >= 0.
// Exact through the 8 corners for max(m) <= 8; beyond, 1/r plus the r^-5 and
// r^-7 terms of the cube average sinh(d/2)/(d/2) applied to the harmonic 1/r.
__device__ double cell_inverse_distance(int mx, int my, int mz) {
  const int mmax = max(mx, max(my, mz));
  if (mmax <= 8) {
    double s = 0.0;
    for (int c = 0; c < 8; ++c) {
      const int sx = c & 1, sy = (c >> 1) & 1, sz = (c >> 2) & 1;
      const double f = prism_antiderivative(mx - 0.5 + sx, my - 0.5 + sy, mz - 0.5 + sz);
      s += ((sx + sy + sz) & 1) ? f : -f;
    }
    return s;
  }
  const double x2 = double(mx) * mx, y2 = double(my) * my, z2 = double(mz) * mz;
  const double r2 = x2 + y2 + z2;
  const double r = sqrt(r2);
  const double s4 = x2 * x2 + y2 * y2 + z2 * z2;
  const double p22 = x2 * y2 + x2 * z2 + y2 * z2;
  const double r4 = r2 * r2;
  const double t4 = (-7.0 / 480.0 * s4 + 7.0 / 160.0 * p22) / (r4 * r4 * r);
  const double s6 = x2 * x2 * x2 + y2 * y2 * y2 + z2 * z2 * z2;
  const double p42 = x2 * x2 * (y2 + z2) + y2 * y2 * (x2 + z2) + z2 * z2 * (x2 + y2);
  const double r12 = r4 * r4 * r4;
  const double t6 = (2.0 * s6 - 15.0 * p42 + 180.0 * x2 * y2 * z2) / 1344.0 / (r12 * r);
  return 1.0 / r + t4 + t6;
}

// ---------------------------------------------------------------------------
// x passes
// ---------------------------------------------------------------------------
template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) void k_xfwd(XParams<T> p) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<T>* buf = reinterpret_cast<cplx<T>*>(smem_raw);
  const int tid = threadIdx.x;
  const int Lx = p.g.Lx, Kx = p.g.Kx, P = p.P, lgP = p.lgP, Lin = p.Lin;
  const int pair0 = blockIdx.x * P;
  cplx<T>* work = p.work;
  const Slot<T> sl = p.tab.s[p.batch.slot[blockIdx.y]];
  double alpha = 0.0;
  bool upd = false;
  if constexpr (MODE == XF_SOLVE) {
    int k;
    XHead<> hd;
    xfwd_head_load(sl, p.n_pap_parts, hd);
    if (!xfwd_head_finish(sl, p.n_pap_parts, hd, &k, &alpha, &upd)) return;
    work = sl.work;
  }
  double mu = 0.0, rr = 0.0;
  for (int e = tid; e < P * Lin; e += kThreads) {
    const int pp = e / Lin;
    const int x = e - pp * Lin;
    const int ra = 2 * (pair0 + pp), rb = ra + 1;
    T a = T(0), b = T(0);
    if constexpr (MODE == XF_SOLVE) {
      if (ra < p.nrows) a = solve_prologue(sl, (size_t)ra * p.in_row_stride + x, upd, alpha, rr);
      if (rb < p.nrows) b = solve_prologue(sl, (size_t)rb * p.in_row_stride + x, upd, alpha, rr);
      mu += double(a) + double(b);
    } else if constexpr (MODE == XF_REAL) {
      if (ra < p.nrows) a = T(p.in_real[(size_t)ra * p.in_row_stride + x]);
      if (rb < p.nrows) b = T(p.in_real[(size_t)rb * p.in_row_stride + x]);
    } else {   // XF_GEN_FREE: K(m) = I(m)/h on the cyclic padded grid
      const int mx = x <= p.g.nx ? x : Lx - x;
      const double inv_h = 1.0 / p.g.h;
      if (ra < p.nrows) {
        const int y = ra % p.rows_per_plane, z = ra / p.rows_per_plane;
        const int my = y <= p.g.ny ? y : p.g.Ly - y, mz = z <= p.g.nz ? z : p.g.Lz - z;
        a = T(cell_inverse_distance(mx, my, mz) * inv_h);
      }
      if (rb < p.nrows) {
        const int y = rb % p.rows_per_plane, z = rb / p.rows_per_plane;
        const int my = y <= p.g.ny ? y : p.g.Ly - y, mz = z <= p.g.nz ? z : p.g.Lz - z;
        b = T(cell_inverse_distance(mx, my, mz) * inv_h);
      }
    }
    buf[(x << lgP) + pp] = cmk(a, b);
  }
  for (int e = tid; e < P * (Lx - Lin); e += kThreads) {
    buf[((Lin + (e >> lgP)) << lgP) + (e & (P - 1))] = cmk(T(0), T(0));
  }
  __syncthreads();
  lds_fft<T, false>(buf, Lx, lgP, p.rp, p.tw);
  for (int e = tid; e < P * Kx; e += kThreads) {
    const int pp = e / Kx;
    const int kk = e - pp * Kx;
    const int ra = 2 * (pair0 + pp), rb = ra + 1;
    const cplx<T> zk = buf[(kk << lgP) + pp];
    const int km = kk == 0 ? 0 : Lx - kk;
    const cplx<T> zm = buf[(km << lgP) + pp];
    const T half = T(0.5);
    const cplx<T> xa = cmk(half * (zk.x + zm.x), half * (zk.y - zm.y));
    const cplx<T> xb = cmk(half * (zk.y + zm.y), half * (zm.x - zk.x));
    if (ra < p.nrows) {
      const size_t o = (size_t)(ra / p.rows_per_plane) * p.plane_stride +
                       (size_t)(ra % p.rows_per_plane) * Kx + kk;
      work[o] = xa;
    }
    if (rb < p.nrows) {
      const size_t o = (size_t)(rb / p.rows_per_plane) * p.plane_stride +
                       (size_t)(rb % p.rows_per_plane) * Kx + kk;
      work[o] = xb;
    }
  }
  if constexpr (MODE == XF_SOLVE) {
    const double s2 = block_sum(rr);
    if (tid == 0) sl.part_rr[blockIdx.x] = s2;
    if (p.periodic_mean) {
      const double s = block_sum(mu);
      if (tid == 0) sl.part_mu[blockIdx.x] = s;
    }
  }
}

template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) void k_xinv(XParams<T> p) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<T>* buf = reinterpret_cast<cplx<T>*>(smem_raw);
  const int tid = threadIdx.x;
  const int Lx = p.g.Lx, Kx = p.g.Kx, P = p.P, lgP = p.lgP, Lout = p.Lout;
  const int pair0 = blockIdx.x * P;
  cplx<T>* work = p.work;
  const Slot<T> sl = p.tab.s[p.batch.slot[blockIdx.y]];
  DirArgs dir{};
  if constexpr (MODE == XI_SOLVE) {
    if (solve_stopped(sl.st)) return;
    work = sl.work;
    dir.fresh = sl.st->fresh;
    dir.beta = sl.st->beta;
    dir.mu = p.periodic_mean ? sl.st->mu : 0.0;
  }
  for (int e = tid; e < P * Kx; e += kThreads) {
    const int pp = e / Kx;
    const int kk = e - pp * Kx;
    const int ra = 2 * (pair0 + pp), rb = ra + 1;
    cplx<T> xa = cmk(T(0), T(0)), xb = cmk(T(0), T(0));
    if (ra < p.nrows)
      xa = work[(size_t)(ra / p.rows_per_plane) * p.plane_stride +
                (size_t)(ra % p.rows_per_plane) * Kx + kk];
    if (rb < p.nrows)
      xb = work[(size_t)(rb / p.rows_per_plane) * p.plane_stride +
                (size_t)(rb % p.rows_per_plane) * Kx + kk];
    if (kk == 0 || 2 * kk == Lx) {   // self-conjugate bins of a real row
      xa.y = T(0);
      xb.y = T(0);
    }
    buf[(kk << lgP) + pp] = cmk(xa.x - xb.y, xa.y + xb.x);          // xa + i xb
    const int km = Lx - kk;
    if (kk > 0 && km >= Kx) buf[(km << lgP) + pp] = cmk(xa.x + xb.y, xb.x - xa.y);
  }
  __syncthreads();
  lds_fft<T, true>(buf, Lx, lgP, p.rp, p.tw);
  const bool per = p.periodic_mean != 0;
  double acc = 0.0;
  for (int e = tid; e < P * Lout; e += kThreads) {
    const int pp = e / Lout;
    const int x = e - pp * Lout;
    const int ra = 2 * (pair0 + pp), rb = ra + 1;
    const cplx<T> z = buf[(x << lgP) + pp];
    if (ra < p.nrows) {
      const size_t o = (size_t)ra * p.in_row_stride + x;
      if constexpr (MODE == XI_SOLVE) solve_epilogue(sl, o, z.x, dir, per, acc);
      else p.out_real[o] = double(z.x);
    }
    if (rb < p.nrows) {
      const size_t o = (size_t)rb * p.in_row_stride + x;
      if constexpr (MODE == XI_SOLVE) solve_epilogue(sl, o, z.y, dir, per, acc);
      else p.out_real[o] = double(z.y);
    }
  }
  if constexpr (MODE == XI_SOLVE) {
    const double s1 = block_sum(acc);
    if (tid == 0) sl.part_pap[blockIdx.x] = s1;
  }
}

// ---------------------------------------------------------------------------
// strided passes (y, z)
// ---------------------------------------------------------------------------
template <typename T, int MODE>
__global__ __launch_bounds__(kThreads) void k_strided(SParams<T> p) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cplx<T>* buf = reinterpret_cast<cplx<T>*>(smem_raw);
  const int tid = threadIdx.x;
  // y inverse of a solve: work-group 0 takes the stop decision, the tiles
  // start at work-group 1
  const int dec = MODE == ST_INV && (p.decide || p.sc.st) ? 1 : 0;
  if (MODE == ST_INV && dec && blockIdx.x == 0) {
    if (p.sc.st) sc_decide_group(p.sc.part, p.sc.nparts, p.sc.st);
    else pcg_decide(p.tab.s[p.batch.slot[blockIdx.y]], p.dec);
    return;
  }
  cplx<T>* work = p.work;
  const SolveState* st = nullptr;
  double* part_delta = nullptr;
  if (work == nullptr) {
    const Slot<T> sl = p.tab.s[p.batch.slot[blockIdx.y]];
    if (solve_stopped(sl.st)) return;
    work = sl.work;
    st = sl.st;
    part_delta = sl.part_delta;
  }
  const int B = p.B, lgB = p.lgB, L = p.L, Lin = p.Lin;
  const int pen0 = (blockIdx.x - dec) * B;
  for (int e = tid; e < (Lin << lgB); e += kThreads) {
    const int b = e & (B - 1);
    const int t = e >> lgB;
    const int pen = pen0 + b;
    cplx<T> v = cmk(T(0), T(0));
    if (pen < p.npencils) {
      const int grp = pen / p.per_group;
      const size_t base = (size_t)grp * p.group_stride + (pen - grp * p.per_group);
      v = work[base + (size_t)t * p.elem_stride];
    }
    buf[e] = v;
  }
  for (int e = tid; e < ((L - Lin) << lgB); e += kThreads) buf[(Lin << lgB) + e] = cmk(T(0), T(0));
  __syncthreads();
  if constexpr (MODE == ST_INV) {
    lds_fft<T, true>(buf, L, lgB, p.rp, p.tw);
  } else {
    lds_fft<T, false>(buf, L, lgB, p.rp, p.tw);
  }
  if constexpr (MODE == ST_CONV) {
    const int Lyh = p.Ly / 2 + 1;
    double dacc = 0.0;              // (v, r) by Parseval, as in the two-level passes
    for (int e = tid; e < (L << lgB); e += kThreads) {
      const int b = e & (B - 1);
      const int t = e >> lgB;
      const int pen = pen0 + b;
      if (pen < p.npencils) {
        const int ky = pen / p.Kx;
        const int kx = pen - ky * p.Kx;
        const int kyf = min(ky, p.Ly - ky);
        const int kzf = min(t, p.Lz - t);
        T m = p.table[((size_t)kzf * Lyh + kyf) * p.Kx + kx];
        if (p.k0_from_slot && pen == 0 && t == 0) m = T(st->g0);
        const cplx<T> w = buf[e];
        dacc += double(half_bin_weight(kx, p.Lx)) * double(m) *
                (double(w.x) * double(w.x) + double(w.y) * double(w.y));
        buf[e] = cscale(w, m);
      }
    }
    if (part_delta) {
      const double sd = block_sum(dacc);
      if (tid == 0) part_delta[blockIdx.x] = sd;
    }
    __syncthreads();
    lds_fft<T, true>(buf, L, lgB, p.rp, p.tw);
  }
  for (int e = tid; e < (p.Lout << lgB); e += kThreads) {
    const int b = e & (B - 1);
    const int t = e >> lgB;
    const int pen = pen0 + b;
    if (pen < p.npencils) {
      const int grp = pen / p.per_group;
      const size_t base = (size_t)grp * p.group_stride + (pen - grp * p.per_group);
      work[base + (size_t)t * p.elem_stride] = buf[e];
    }
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Work-groups of the generic x passes (also the count of their partials).
template <typename T> static int generic_xpass_groups(const XParams<T>& p) {
  const int npairs = (p.nrows + 1) / 2;
  return (npairs + p.P - 1) / p.P;
}

// Partials of the solve-mode x passes: one per wavefront in the two-level
// passes, one per work-group in the generic ones.
template <typename T> int xpass_parts(const XParams<T>& p) {
  if (fast_solve(p)) return fast_xpass_parts<T>(p.g.Lx, p.nrows);
  return generic_xpass_groups(p);
}

template <typename T> void launch_xfwd(int mode, const XParams<T>& p, hipStream_t s) {
  if (p.sh.N > 0) {                    // the generic passes know no planes
    if (!fast_length(p.g.Lx) || !fast_xfwd<T>(mode, p, s))
      throw DevError{hipErrorInvalidConfiguration};
    return;
  }
  if (mode != XF_GEN_FREE && fast_length(p.g.Lx) && fast_xfwd<T>(mode, p, s)) return;
  const dim3 grid(generic_xpass_groups(p), p.has_slots ? p.batch.n : 1);
  const size_t lds = (size_t)p.P * p.g.Lx * sizeof(cplx<T>);
  if (mode == XF_SOLVE) GPS_LAUNCH((k_xfwd<T, XF_SOLVE>), grid, dim3(kThreads), lds, s, p);
  else if (mode == XF_REAL) GPS_LAUNCH((k_xfwd<T, XF_REAL>), grid, dim3(kThreads), lds, s, p);
  else GPS_LAUNCH((k_xfwd<T, XF_GEN_FREE>), grid, dim3(kThreads), lds, s, p);
}

template <typename T> void launch_xinv(int mode, const XParams<T>& p, hipStream_t s) {
  if (p.sh.N > 0) {
    if (!fast_length(p.g.Lx) || !fast_xinv<T>(mode, p, s))
      throw DevError{hipErrorInvalidConfiguration};
    return;
  }
  if (fast_length(p.g.Lx) && fast_xinv<T>(mode, p, s)) return;
  const dim3 grid(generic_xpass_groups(p), p.has_slots ? p.batch.n : 1);
  const size_t lds = (size_t)p.P * p.g.Lx * sizeof(cplx<T>);
  if (mode == XI_SOLVE) GPS_LAUNCH((k_xinv<T, XI_SOLVE>), grid, dim3(kThreads), lds, s, p);
  else GPS_LAUNCH((k_xinv<T, XI_REAL>), grid, dim3(kThreads), lds, s, p);
}

template <typename T> int strided_parts(const SParams<T>& p) {
  if (fast_length(p.L)) return fast_strided_parts<T>(p);
  return (p.npencils + p.B - 1) / p.B;
}

template <typename T> void launch_strided(int mode, const SParams<T>& p, hipStream_t s) {
  if (fast_length(p.L) && fast_strided<T>(mode, p, s)) return;
  const int dec = mode == ST_INV && (p.decide || p.sc.st) ? 1 : 0;   // the decision work-group
  const dim3 grid((p.npencils + p.B - 1) / p.B + dec, p.work ? 1 : p.batch.n);
  const size_t lds = (size_t)p.B * p.L * sizeof(cplx<T>);
  if (mode == ST_FWD) GPS_LAUNCH((k_strided<T, ST_FWD>), grid, dim3(kThreads), lds, s, p);
  else if (mode == ST_INV) GPS_LAUNCH((k_strided<T, ST_INV>), grid, dim3(kThreads), lds, s, p);
  else GPS_LAUNCH((k_strided<T, ST_CONV>), grid, dim3(kThreads), lds, s, p);
}

// ---------------------------------------------------------------------------
// plane pass
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_plane_table(PlaneShape sh, const double* __restrict__ t64, int Kx, int Ly,
                              T* __restrict__ out) {
  const int Lyh = Ly / 2 + 1, Lzh = sh.Lz / 2 + 1;
  const long long n = (long long)Kx * kPlaneParts * Lzh * sh.N;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const int pos = (int)(i % sh.N);
    const int kz = (int)((i / sh.N) % Lzh);
    const int t = (int)(i / ((long long)sh.N * Lzh));
    const int kx = t / kPlaneParts, r = t - kx * kPlaneParts;
    const int a = pos / sh.A2, b = pos - a * sh.A2;      // k' = a + A1 b
    const int ky = r + kPlaneParts * (a + sh.A1 * b);
    out[i] = T(t64[((size_t)kz * Lyh + min(ky, Ly - ky)) * Kx + kx]);
  }
}

template <typename T>
void launch_plane_table(const PlaneShape& sh, const double* t64, int Kx, int Ly, T* out,
                        hipStream_t s) {
  const long long n = (long long)Kx * Ly * (sh.Lz / 2 + 1);
  const int grid = (int)std::min<long long>((n + kThreads - 1) / kThreads, 65535);
  GPS_LAUNCH((k_plane_table<T>), dim3(grid), dim3(kThreads), 0, s, sh, t64, Kx, Ly, out);
}
template void launch_plane_table<float>(const PlaneShape&, const double*, int, int, float*,
                                        hipStream_t);
template void launch_plane_table<double>(const PlaneShape&, const double*, int, int, double*,
                                         hipStream_t);

static bool plane_radix(int r) {
  return (r >= 2 && r <= 10) || r == 12 || r == 14 || r == 15 || r == 16;
}

// n = a b over the codelets of the plane pass (b = 1 for n <= 5), the larger
// factor as small as possible.  Along z (even: a padded axis) a is the larger, and
// even; along y b is, the run of a row that neighbouring lanes load and store.
static bool plane_split(int n, bool along_z, bool even, int* a, int* b) {
  int best = 17;
  for (int x = 2; x <= 16; ++x) {
    if (n % x || !plane_radix(x) || (even && x % 2)) continue;
    const int y = n / x;
    if (y == 1 ? n > 5 : !plane_radix(y)) continue;
    const int m = std::max(x, y);
    if (m < best || (m == best && along_z)) {
      best = m;
      *a = x;
      *b = y;
    }
  }
  return best < 17;
}

// Dynamic LDS of the plane kernels: a CU's 160 KB less their static words.
constexpr int kPlaneLds = 160 * 1024 - 512;

// The plane pass runs where its tile fits one work-group's LDS (FP32: cubes up to
// 98^3 free and wire, 180^3 periodic; FP64: 63^3 free, 98^3 wire, 128^3 periodic), where the
// work-groups are many enough for their size, and on grids small enough that
// its launches and transposes count.  Measured against the y, z, y passes, x the
// time of the latter over the former:
//   lds <= 1100 per group    70 random grids of 18 to 120 points 1.01 to 1.20 on this
//                            side (two FP64 grids at 0.996), 0.97 beyond it (FP64, 105 x 108
//                            x 70 periodic: 72 groups of 96 KB; 96^3 surface: 98 of 150 KB)
//   n <= 5e6                 vacuum solves (FP32 and FP64) of 69 grids of 0.3 to 4.8 million
//                            points: 1.02 to 1.23; of four beyond: 0.98 to 1.02
// PCG solves (FP32 alone, see use_plane in gps_api.hip) carry the direction update
// in the x inverse, which beside the plane pass takes more registers and, on a large grid, more
// of the iteration than the transposes:
//   n <= 1.5e6               45 grids: 1.01 to 1.24
//   n <= 3.5e6               where a thread of the x inverse holds at most 209 values (its
//                            kernel 254 VGPRs, two wavefronts per SIMD): 53 grids, 0.99 to 1.23,
//                            mean 1.07; where it holds more (periodic x lengths 81, 100, 108,
//                            120, 144, 168, 180, 196): eight grids, 0.90 to 0.98
//   beyond                   16 grids of 3.6 to 7.5 million points: 0.85 to 1.03, mean 0.96
constexpr long long kPlanePoints = 5000000, kPlaneSolvePoints = 3500000, kPlaneFewPoints = 1500000;
constexpr int kPlaneSolveValues = 209;

PlaneShape plane_shape(const Geom& g, size_t elem) {
  PlaneShape none{};
  const long long n = (long long)g.nx * g.ny * g.nz;
  if (!fast_length(g.Lx) || g.Lx > kPlaneMaxLx || g.Ly % kPlaneParts || n > kPlanePoints)
    return none;
  PlaneShape s{};
  s.nz = g.nz;
  s.ny = g.ny;
  s.Lz = g.Lz;
  s.N = g.Ly / kPlaneParts;
  s.nm = g.ny / s.N;
  s.padz = !g.periodic_z;
  if (s.N < 2 || !plane_split(s.N, false, false, &s.A1, &s.A2) ||
      !plane_split(s.Lz, true, s.padz, &s.C1, &s.C2) || s.C2 == 1)
    return none;
  s.PY = s.N | 1;                     // odd: the y steps' lanes run over z
  s.lds = ((size_t)s.PY * s.Lz + s.Lz + 2 * s.N) * 2 * elem;
  if (s.lds > (size_t)kPlaneLds || s.lds > 1100 * (size_t)plane_groups(g.Kx)) return none;
  const int periodic = g.periodic_x && g.periodic_y && g.periodic_z;
  s.solve = elem == sizeof(float) && n <= kPlaneSolvePoints &&
            (n <= kPlaneFewPoints || fast_xinv_values(g.Lx, g.nx, periodic) <= kPlaneSolveValues);
  // threads: the count whose four kinds of steps take the fewest rounds, weighed
  // by their lengths and about 8 more for a step's fixed work
  const int jobs[4] = {s.nz * s.A2, s.nz * s.A1, s.N * s.C2, s.N * s.C1};
  const int len[4] = {s.A1, s.A2, s.C1, s.C2};
  double best = 1e30;
  for (int nt = 64; nt <= plane_threads(elem); nt += 64) {
    double cost = 0.002 * nt;
    for (int i = 0; i < 4; ++i) cost += (double)((jobs[i] + nt - 1) / nt) * (len[i] + 8);
    if (cost < best) {
      best = cost;
      s.threads = nt;
    }
  }
  s.div_A2 = make_fastdiv((unsigned)s.A2);
  s.div_nz = make_fastdiv((unsigned)s.nz);
  s.div_N = make_fastdiv((unsigned)s.N);
  s.div_ny = make_fastdiv((unsigned)s.ny);
  return s;
}

void plane_allow_lds() {
  const void* kernels[] = {
      reinterpret_cast<const void*>(&k_plane<float, true>),
      reinterpret_cast<const void*>(&k_plane<float, false>),
      reinterpret_cast<const void*>(&k_plane<double, true>),
      reinterpret_cast<const void*>(&k_plane<double, false>)};
  for (const void* k : kernels)
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kPlaneLds) != hipSuccess)
      (void)hipGetLastError();
}

template <typename T> void launch_plane(const PlaneParams<T>& p, hipStream_t s) {
  if (sizeof(T) != sizeof(float) && !p.work) throw DevError{hipErrorInvalidConfiguration};
  const dim3 grid(plane_groups(p.Kx) + (p.sc.st ? 1 : 0), p.work ? 1 : p.batch.n);
  const dim3 blk(p.sh.threads);
  if (p.sh.padz) GPS_LAUNCH((k_plane<T, true>), grid, blk, p.sh.lds, s, p);
  else GPS_LAUNCH((k_plane<T, false>), grid, blk, p.sh.lds, s, p);
}
template void launch_plane<float>(const PlaneParams<float>&, hipStream_t);
template void launch_plane<double>(const PlaneParams<double>&, hipStream_t);

template int strided_parts<float>(const SParams<float>&);
template int strided_parts<double>(const SParams<double>&);
template int xpass_parts<float>(const XParams<float>&);
template int xpass_parts<double>(const XParams<double>&);
template void launch_xfwd<float>(int, const XParams<float>&, hipStream_t);
template void launch_xfwd<double>(int, const XParams<double>&, hipStream_t);
template void launch_xinv<float>(int, const XParams<float>&, hipStream_t);
template void launch_xinv<double>(int, const XParams<double>&, hipStream_t);
template void launch_strided<float>(int, const SParams<float>&, hipStream_t);
template void launch_strided<double>(int, const SParams<double>&, hipStream_t);

}  // namespace gps
