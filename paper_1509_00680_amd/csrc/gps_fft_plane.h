// Plane pass: the y forward, z and y inverse passes of the vacuum solver in one
// launch, for planes that fit LDS.
//
// The x forward pass leaves its half spectrum as one plane per kx, row-major in
// the grid's rows: half[kx][z][y].  A work-group takes one kx and one parity r of
// ky (ky = r + 2 k'), so its y transform has length N = Ly/2:
//   fold     x_r[j] = w_Ly^(r j) (x[j] + (-1)^r x[j + N]),  j < N
//            (a padded y axis holds no data at j >= N: nm = 1 block, not 2)
//   y        N-point DFT over j, for the nz rows of the plane
//   z        Lz-point DFT (nz data points), times the Green's spectrum, inverse
//   y        inverse N-point DFT, times w_Ly^(-r j)
// and leaves the partial sum Y_r[z][j] in work[kx][r][z][j]; the x inverse pass
// adds the parities: out[j] = Y_0 + Y_1, out[j + N] = Y_0 - Y_1.  Two parities
// halve the tile and double the work-groups; finer residues were slower (96^3
// FP32: 26.8 us at four against 22.0, and the x inverse reads them all).
//
// Both transforms are two-level and in place in one LDS tile: the first factor's
// DFTs write their outputs where their inputs lay (element A2 k1 + n2), the
// second factor's then leave X[k1 + A1 k2] at A2 k1 + k2, and the inverse goes
// back the same way, so no step needs a second tile or a barrier between its
// reads and its writes, and the z pass keeps the second factor's values in
// registers from the forward transform over the multiplication to the inverse.
//
// Bound by the latency of its seven steps, over few work-groups: 50 on 256 CUs at 24^3, 66
// at 32^3, 194 at 96^3 (of 152 KB LDS, so at most one per CU).  It wins by the launches
// and the transposes through memory that it saves.  Plans with and without it in turn, one
// MI355X: mixed solves at 1e-6 of 32^3 1095 -> 976 us, 64^3 1655 -> 1486, 96^3 3848 -> 3555 (kernels
// 29.4 -> 20.0 us an iteration, the x inverse + 3.5), vacuum solve 24^3 FP64 29.7 -> 26.4 us, SC
// 60^3 FP64 1953 -> 1892 us.  Errors against FP64, over those of the three passes: FP32 vacuum
// solves 0.975 to 1.035, mean 1.006 (12 grids, 30 solutes each), mixed solves 0.92 to
// 1.04, mean 1.008: the fold's extra twiddle product is no more than their scatter.
#pragma once

#include <cstdint>

#include "gps_fft_reg.h"
#include "gps_iter.h"
#include "gps_launch.h"
#include "gps_sc.h"

namespace gps {

// Calls f with the codelet length R as a compile-time constant.
template <typename F>
__device__ __forceinline__ void with_radix(int R, F&& f) {
  switch (R) {
#define GPS_R(N) case N: f(std::integral_constant<int, N>{}); return;
    GPS_R(2) GPS_R(3) GPS_R(4) GPS_R(5) GPS_R(6) GPS_R(7) GPS_R(8) GPS_R(9) GPS_R(10)
    GPS_R(12) GPS_R(14) GPS_R(15) GPS_R(16)
#undef GPS_R
    default: break;
  }
}

// PADZ: the pencils along z hold Lz/2 points (the zero half is compile time).
template <typename T, bool PADZ>
__global__ __launch_bounds__(plane_threads(sizeof(T))) void k_plane(PlaneParams<T> p) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int tid = threadIdx.x, NT = blockDim.x;
  const int dec = p.sc.st ? 1 : 0;                // the tiles start at work-group 1
  if (dec && blockIdx.x == 0) {
    sc_decide_group(p.sc.part, p.sc.nparts, p.sc.st);
    return;
  }
  // copies: a parameter struct referenced by the lambdas would be moved to
  // scratch memory
  const int nz = p.sh.nz, ny = p.sh.ny, N = p.sh.N, PY = p.sh.PY, nm = p.sh.nm;
  const int A1 = p.sh.A1, A2 = p.sh.A2, C1 = p.sh.C1, C2 = p.sh.C2, Lz = p.sh.Lz;
  const FastDiv div_A2 = p.sh.div_A2, div_nz = p.sh.div_nz, div_N = p.sh.div_N;
  const cplx<T>* const ptwy = p.twy;
  const cplx<T>* const ptwz = p.twz;
  const T* const table = p.table;
  const int k0_from_slot = p.k0_from_slot;
  cplx<T>* tile = reinterpret_cast<cplx<T>*>(smem_raw);
  cplx<T>* twz = tile + (size_t)PY * Lz;          // w_Lz^i
  cplx<T>* twy = twz + Lz;                        // w_N^i
  cplx<T>* fold = twy + N;                        // w_Ly^i (used for r = 1)
  const cplx<T>* half = p.half;
  cplx<T>* work = p.work;
  const SolveState* st = nullptr;
  double* part_delta = nullptr;
  // PCG solves: FP32 alone (launch_plane refuses FP64; without this branch the
  // FP64 kernel holds 185 VGPRs and 90 spilled SGPRs, with it 179 and 73: 24^3 26.2
  // against 25.7 us)
  if (work == nullptr) {
    const Slot<T> sl = p.tab.s[p.batch.slot[blockIdx.y]];
    half = sl.half;
    work = sl.work;
    st = sl.st;
    part_delta = sl.part_delta;
    if (solve_stopped(st)) return;
  }
  const int t = xcd_tile(blockIdx.x, gridDim.x) - dec;   // the two of one kx meet in one L2
  const int kx = t >> 1, r = t & 1;
  const cplx<T>* src = half + (size_t)kx * nz * ny;
  cplx<T>* dst = work + (size_t)t * nz * N;

  // ---- fold and first factor along y, from memory to LDS ----
  with_radix(A1, [&](auto RC) __attribute__((always_inline)) {
    constexpr int R = decltype(RC)::value;
    const int jobs = nz * A2;
    bool staged = false;
    for (int job = tid; job < jobs || !staged; job += NT) {
      const int jc = min(job, jobs - 1);
      const int z = (int)fast_div((unsigned)jc, div_A2), n2 = jc - z * A2;
      cplx<T> x[R];
      const cplx<T>* s0 = src + z * ny + n2;
#pragma unroll
      for (int i = 0; i < R; ++i) x[i] = s0[A2 * i];
      if (nm == 2) {
        cplx<T> v[R];
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = s0[N + A2 * i];
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = r ? csub(x[i], v[i]) : cadd(x[i], v[i]);
      }
      if (!staged) {
        for (int i = tid; i < Lz; i += NT) twz[i] = ptwz[i];
        for (int i = tid; i < N; i += NT) {
          twy[i] = ptwy[2 * i];
          fold[i] = ptwy[i];
        }
        __syncthreads();
        staged = true;
      }
      if (job < jobs) {
        if (r > 0) {
#pragma unroll
          for (int i = 0; i < R; ++i) x[i] = cmul(x[i], fold[A2 * i + n2]);
        }
        reg_fft<T, false, R>(x);
        cplx<T>* d = tile + z * PY + n2;
        d[0] = x[0];
#pragma unroll
        for (int k = 1; k < R; ++k) d[A2 * k] = A2 > 1 ? cmul(x[k], twy[n2 * k]) : x[k];
      }
    }
  });
  __syncthreads();
  // ---- second factor along y, in place ----
  if (A2 > 1) {
    with_radix(A2, [&](auto RC) __attribute__((always_inline)) {
      constexpr int R = decltype(RC)::value;
      for (int job = tid; job < nz * A1; job += NT) {
        const int k1 = (int)fast_div((unsigned)job, div_nz), z = job - k1 * nz;
        cplx<T>* d = tile + z * PY + R * k1;
        cplx<T> x[R];
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = d[i];
        reg_fft<T, false, R>(x);
#pragma unroll
        for (int i = 0; i < R; ++i) d[i] = x[i];
      }
    });
    __syncthreads();
  }
  // ---- first factor along z, in place (zero half pruned) ----
  with_radix(C1, [&](auto RC) __attribute__((always_inline)) {
    constexpr int R = decltype(RC)::value;
    if constexpr (!PADZ || R % 2 == 0) {
      for (int job = tid; job < N * C2; job += NT) {
        const int q = (int)fast_div((unsigned)job, div_N), y = job - q * N;
        cplx<T>* d = tile + q * PY + y;
        const int step = C2 * PY;
        cplx<T> x[R];
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = PADZ && i >= R / 2 ? cmk(T(0), T(0)) : d[i * step];
        reg_fft<T, false, R>(x);
        d[0] = x[0];
#pragma unroll
        for (int k = 1; k < R; ++k) d[k * step] = cmul(x[k], twz[q * k]);
      }
    }
  });
  __syncthreads();
  // ---- second factor along z, Green's spectrum, and back ----
  double dacc = 0.0;
  with_radix(C2, [&](auto RC) __attribute__((always_inline)) {
    constexpr int R = decltype(RC)::value;
    const T* const tt = table + (size_t)t * (Lz / 2 + 1) * N;
    for (int job = tid; job < N * C1; job += NT) {
      const int k1 = (int)fast_div((unsigned)job, div_N), y = job - k1 * N;
      T gm[R];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int kz = k1 + C1 * i;
        gm[i] = tt[min(kz, Lz - kz) * N + y];
      }
      if (k0_from_slot && t == 0 && job == 0) gm[0] = T(st->g0);
      cplx<T>* d = tile + (R * k1) * PY + y;
      cplx<T> x[R];
#pragma unroll
      for (int i = 0; i < R; ++i) x[i] = d[i * PY];
      reg_fft<T, false, R>(x);
      double ws = 0.0;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const cplx<T> w = x[i];
        x[i] = cscale(w, gm[i]);
        ws += double(x[i].x) * double(w.x) + double(x[i].y) * double(w.y);
      }
      dacc += ws;
      reg_fft<T, true, R>(x);
      d[0] = x[0];
#pragma unroll
      for (int i = 1; i < R; ++i) {
        const cplx<T> w = twz[i * k1];
        d[i * PY] = cmul(x[i], cmk(w.x, -w.y));
      }
    }
  });
  __syncthreads();
  with_radix(C1, [&](auto RC) __attribute__((always_inline)) {
    constexpr int R = decltype(RC)::value;
    if constexpr (!PADZ || R % 2 == 0) {
      for (int job = tid; job < N * C2; job += NT) {
        const int q = (int)fast_div((unsigned)job, div_N), y = job - q * N;
        cplx<T>* d = tile + q * PY + y;
        const int step = C2 * PY;
        cplx<T> x[R];
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = d[i * step];
        reg_fft<T, true, R>(x);
#pragma unroll
        for (int i = 0; i < (PADZ ? R / 2 : R); ++i) d[i * step] = x[i];
      }
    }
  });
  __syncthreads();
  // ---- back along y ----
  if (A2 > 1) {
    with_radix(A2, [&](auto RC) __attribute__((always_inline)) {
      constexpr int R = decltype(RC)::value;
      for (int job = tid; job < nz * A1; job += NT) {
        const int k1 = (int)fast_div((unsigned)job, div_nz), z = job - k1 * nz;
        cplx<T>* d = tile + z * PY + R * k1;
        cplx<T> x[R];
#pragma unroll
        for (int i = 0; i < R; ++i) x[i] = d[i];
        reg_fft<T, true, R>(x);
        d[0] = x[0];
#pragma unroll
        for (int i = 1; i < R; ++i) {
          const cplx<T> w = twy[i * k1];
          d[i] = cmul(x[i], cmk(w.x, -w.y));
        }
      }
    });
    __syncthreads();
  }
  with_radix(A1, [&](auto RC) __attribute__((always_inline)) {
    constexpr int R = decltype(RC)::value;
    for (int job = tid; job < nz * A2; job += NT) {
      const int z = (int)fast_div((unsigned)job, div_A2), n2 = job - z * A2;
      const cplx<T>* d = tile + z * PY + n2;
      cplx<T> x[R];
#pragma unroll
      for (int i = 0; i < R; ++i) x[i] = d[A2 * i];
      reg_fft<T, true, R>(x);
      cplx<T>* o = dst + z * N + n2;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if (r > 0) {
          const cplx<T> w = fold[A2 * i + n2];
          x[i] = cmul(x[i], cmk(w.x, -w.y));
        }
        __builtin_nontemporal_store(x[i].x, &o[A2 * i].x);
        __builtin_nontemporal_store(x[i].y, &o[A2 * i].y);
      }
    }
  });
  if (part_delta) {                               // one partial per work-group
    const double sd = block_sum(dacc);
    if (tid == 0) part_delta[t] = sd * double(half_bin_weight(kx, p.Lx));
  }
}

}  // namespace gps
