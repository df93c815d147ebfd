// Two-level FFT passes: kernels and the launches of one pencil length.
//
// A length L = L1 * L2 transform of a tile of pencils runs as
//   forward:  x[L2 n1 + n2] --(L1-point DFT over n1, in registers)--> Y[n2][k1]
//             Y *= w_L^(n2 k1); one exchange through LDS;
//             (L2-point DFT over n2, in registers) --> X[k1 + L1 k2]
//   inverse:  X[k1 + L1 k2] --(L2-point inverse DFT over k2)--> Z[k1][n_a]
//             Z *= w_L^(-n_a k1); one exchange through LDS;
//             (L1-point inverse DFT over k1) --> x[n_a + L2 n_b]
// so a pass touches LDS once per direction instead of once per radix stage.
// The z pass keeps the spectrum in registers between the forward transform,
// the multiplication by the Green's spectrum and the inverse transform.
//
// Strided (y, z) passes load and store directly between HBM and registers:
// a thread owns one column of one pencil, threads of a wavefront cover B
// adjacent pencils, so every row access is a contiguous B-element segment.
// The x passes stage rows through LDS to keep their loads and stores
// contiguous along x.
#pragma once

#include "gps_fft_reg.h"
#include "gps_iter.h"
#include "gps_launch.h"
#include "gps_sc.h"

namespace gps {

template <typename T> struct FastTile;
template <> struct FastTile<float> { static constexpr int B = 16; };
template <> struct FastTile<double> { static constexpr int B = 8; };
// Pencils per tile of a strided pass: FastTile<T>::B, except for FP32 passes
// of length 320 and 384, which take 8.  Their 16-pencil LDS tile (L x 17
// values, 46-55 KB) fits 2-3 work-groups per CU; the 8-pencil tile fits 5-6,
// which hides more of the latency of the transforms (160^3: z pass 52.5 ->
// 41.5 us, y passes 23.8 / 22.4 -> 21.7 / 21.8 us; 128 x 128 x 192 slab, z
// length 384: 22.3 -> 16.2 us).  At the shorter lengths the 16-pencil tile
// already fits 4 or more, and its 128-byte rows are whole cache lines.
template <typename T> constexpr int strided_tile(int L) {
  return (L >= 320 && FastTile<T>::B == 16) ? 8 : FastTile<T>::B;
}
constexpr int round64(int v) { return (v + 63) / 64 * 64; }
constexpr int larger(int a, int b) { return a > b ? a : b; }
// The tuned lengths keep their first constants (Roots2Pi); the others take the nearest.
constexpr bool kept_roots(int L) {
  return L == 32 || L == 48 || L == 64 || L == 96 || L == 128 || L == 192 || L == 256 ||
         L == 320 || L == 384;
}

// The passes address their buffers with 32-bit byte offsets, and multiply a stride by a
// small count with a 24-bit product.  One axis has at most kMaxFastLen points, the others
// kMaxLen, so the largest buffers (FP64 half spectra, with the short axis along x or not, and
// FP64 fields) stay below 4 GiB and the z pass's strides below 2^24.
constexpr long long kMaxOffset = 1ll << 32;
static_assert(16ll * kMaxLen * kMaxFastLen * (kMaxLen / 2 + 1) <= kMaxOffset, "work buffer");
static_assert(16ll * kMaxLen * kMaxLen * (kMaxFastLen / 2 + 1) <= kMaxOffset, "work buffer");
static_assert(8ll * kMaxLen * kMaxLen * kMaxFastLen <= kMaxOffset, "field");
static_assert(16ll * kMaxLen * (kMaxLen / 2 + 1) < (1 << 24), "stride of the z pass");
static_assert(8ll * (kMaxLen / 2 + 1) * (kMaxLen / 2 + 1) < (1 << 24), "stride of its table");

template <typename T>
__device__ __forceinline__ cplx<T> cconj(cplx<T> a) { return cmk(a.x, -a.y); }

// Load by components: a complex FP64 value copied as a whole into an array that
// lives across a branch is given a stack slot (a wait for the load, a store to
// scratch memory and a second load), its two parts are not.
template <typename T>
__device__ __forceinline__ cplx<T> load_parts(const cplx<T>* p) { return cmk(p->x, p->y); }

// Store of a value that the next kernel reads on other XCDs (the transposes
// around the z pass): non-temporal, so the line does not stay dirty in this
// XCD's L2 until the end-of-kernel write-back.  Large outputs of the y-forward
// and z passes (plain_store: 32 MiB and more, 66 MB at 160^3) are stored
// plainly instead: they then stay in the last-level cache for the next pass
// (160^3: z pass 57.8 -> 52.5 us after a plain y forward; y inverse 25.3 ->
// 22.3 us after a plain z pass).
template <typename T>
__device__ __forceinline__ void store_stream(cplx<T>* dst, cplx<T> v) {
  __builtin_nontemporal_store(v.x, &dst->x);
  __builtin_nontemporal_store(v.y, &dst->y);
}

// ---------------------------------------------------------------------------
// strided passes
// ---------------------------------------------------------------------------
// A work-group transforms NTILE adjacent tiles of B pencils.  Every global load
// of all its tiles is issued first, so the later tiles' loads are in flight
// while the first tile is transformed.  PAD: the pencil holds L/2 data points
// (Hockney zero padding): the forward and z passes read, and the inverse and z
// passes write, only the first L/2 elements, and the zero half is a
// compile-time constant.
template <typename T, int L1, int L2, int MODE, bool PAD, int NTILE, int B, int PLAIN>
__global__ __launch_bounds__(round64(B * larger(L1, L2)))
void k_fstrided(SParams<T> p) {
  constexpr int L = L1 * L2;
  constexpr int PITCH = B + 1;
  constexpr int NT = round64(B * larger(L1, L2));
  __shared__ cplx<T> lds[L * PITCH];
  __shared__ cplx<T> twl[L];
  const int tid = threadIdx.x;
  // y inverse of a solve: work-group 0 only takes the stop decision (it runs
  // beside the transforms instead of after one); the tiles are numbered from
  // work-group 1 on
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
    work = sl.work;
    st = sl.st;
    part_delta = sl.part_delta;
  }
  // twiddles first, then the tile, then the stop flag: all in flight together
  cplx<T> twv[(L + NT - 1) / NT];
#pragma unroll
  for (int i = 0; i < (L + NT - 1) / NT; ++i)
    twv[i] = load_parts(&p.tw[min(tid + i * NT, L - 1)]);   // clamped: no branch around the load
  const int b = tid & (B - 1);
  const int q = tid / B;
  // (xcd_tile maps work-group 0 to tile 0, so the shift keeps every XCD's
  // tiles contiguous)
  const int tile0 = (xcd_tile(blockIdx.x, gridDim.x) - dec) * NTILE;
  // 32-bit byte offsets (checked beside kMaxOffset)
  constexpr unsigned CB = sizeof(cplx<T>);
  const unsigned es = CB * (unsigned)p.elem_stride;
  // Element e of this thread's pencil sits at base + e * es.  Every element a
  // thread touches has e = q + L1 k or e = q + L2 k (k compile-time), so its
  // offset is qb + k * (L1 es) or qb + k * (L2 es): one per-thread product
  // (es < 2^24) and scalar steps.
  const unsigned s1 = (unsigned)L1 * es, s2 = (unsigned)L2 * es;
  int pen[NTILE];
  bool pv[NTILE];
  unsigned base[NTILE], qb[NTILE];
#pragma unroll
  for (int t = 0; t < NTILE; ++t) {
    pen[t] = (tile0 + t) * B + b;
    pv[t] = pen[t] < p.npencils;
    base[t] = 0;
    if (pv[t]) {
      const unsigned grp = fast_div((unsigned)pen[t], p.div_group);
      base[t] = CB * (grp * (unsigned)p.group_stride + ((unsigned)pen[t] - grp * (unsigned)p.per_group));
    }
    qb[t] = base[t] + __umul24((unsigned)q, es);
  }
  // data extents: PAD bounds the input of the forward and z passes and the
  // output of the inverse and z passes
  const int lin = (PAD && MODE != ST_INV) ? L / 2 : p.Lin;
  const int lout = (PAD && MODE != ST_FWD) ? L / 2 : p.Lout;

  // ---- phase 1: every load of every tile (the stop flag is read after them,
  // so both travel together: a stopped solve wastes the loads, never a round
  // trip) ----
  cplx<T> xin[MODE != ST_INV ? NTILE : 1][L1];
  cplx<T> yin[MODE == ST_INV ? NTILE : 1][L2];
  T gm[MODE == ST_CONV ? NTILE : 1][MODE == ST_CONV ? L2 : 1];
  T gw[NTILE];                                  // z pass: half-spectrum weight of the pencil
#pragma unroll
  for (int t = 0; t < NTILE; ++t) {
    if constexpr (MODE != ST_INV) {
      if (q < L2) {
#pragma unroll
        for (int n1 = 0; n1 < L1; ++n1) {
          // branch-free: a clamped element (base 0 for pencils past the end)
          // is loaded and then selected, so the loads issue back to back
          const int e = L2 * n1 + q;
          if (PAD && n1 >= L1 / 2) {
            xin[t][n1] = cmk(T(0), T(0));
          } else if (PAD) {
            // no select: a lane past the last pencil (offset 0) transforms
            // real data and stores nothing
            xin[t][n1] = at_bytes(work, qb[t] + (unsigned)n1 * s2);
          } else {
            // clamped to element lin - 1 (branch-free)
            const unsigned o = e < lin ? qb[t] + (unsigned)n1 * s2 : base[t] + (unsigned)(lin - 1) * es;
            const cplx<T> v = at_bytes(work, o);
            xin[t][n1] = (pv[t] && e < lin) ? v : cmk(T(0), T(0));
          }
        }
      }
      if constexpr (MODE == ST_CONV) {
        // spectrum multipliers of the z pass: prefetched with the tile
        {
          // branch-free: a lane past the last pencil reads pencil 0's entries,
          // and a thread with q >= L1 (NT is B * L1 rounded up to a wavefront)
          // reads those of q = 0; neither is used
          const int Lyh = p.Ly / 2 + 1;
          const int pc = pv[t] ? pen[t] : 0;
          const int qc = q < L1 ? q : 0;
          const int ky = (int)fast_div((unsigned)pc, p.div_kx);
          const int kx = pc - ky * p.Kx;
          gw[t] = T(half_bin_weight(kx, p.Lx));
          const int kyf = min(ky, p.Ly - ky);
          const unsigned row = (unsigned)sizeof(T) * (unsigned)(kyf * p.Kx + kx);
          const unsigned zs = (unsigned)sizeof(T) * (unsigned)(Lyh * p.Kx);
          // folded index min(kz, L - kz) of kz = qc + L1 k2: two arithmetic
          // progressions in k2 and a select (zs < 2^24)
          const unsigned up = row + __umul24((unsigned)qc, zs);
          const unsigned down = row + __umul24((unsigned)(L - qc), zs);
          const unsigned zstep = (unsigned)L1 * zs;
#pragma unroll
          for (int k2 = 0; k2 < L2; ++k2) {
            const unsigned o = qc <= L / 2 - L1 * k2 ? up + (unsigned)k2 * zstep
                                                      : down - (unsigned)k2 * zstep;
            gm[t][k2] = at_bytes(p.table, o);
          }
        }
      }
    } else {
      if (q < L1) {
#pragma unroll
        for (int k2 = 0; k2 < L2; ++k2) {
          const int kk = q + L1 * k2;
          if (PAD) {
            // full-length input (kk < L): no select, as above
            yin[t][k2] = at_bytes(work, qb[t] + (unsigned)k2 * s1);
          } else {
            // clamped to element lin - 1 (branch-free, as above)
            const unsigned o = kk < lin ? qb[t] + (unsigned)k2 * s1 : base[t] + (unsigned)(lin - 1) * es;
            const cplx<T> v = at_bytes(work, o);
            yin[t][k2] = (pv[t] && kk < lin) ? v : cmk(T(0), T(0));
          }
        }
      }
    }
  }
  const int flag = st ? stop_flag_issue(st) : 0;
#pragma unroll
  for (int i = 0; i < (L + NT - 1) / NT; ++i)
    if (tid + i * NT < L) twl[tid + i * NT] = cmk(twv[i].x, twv[i].y);
  if (stop_flag_set(flag)) return;
  __syncthreads();
  const cplx<T>* tw = twl;

  // ---- phase 2: transform the tiles one after the other ----
  double dacc = 0.0;                            // z pass: this thread's part of (v, r)
#pragma unroll
  for (int t = 0; t < NTILE; ++t) {
    if (t > 0) __syncthreads();                 // previous tile's LDS reads are done
    cplx<T> y[L2];
    if constexpr (MODE != ST_INV) {
      if (q < L2) {
        cplx<T> x[L1];
#pragma unroll
        for (int n1 = 0; n1 < L1; ++n1) x[n1] = xin[t][n1];
        reg_fft<T, false, L1, kept_roots(L1 * L2)>(x);
#pragma unroll
        for (int k1 = 1; k1 < L1; ++k1) x[k1] = cmul(x[k1], tw[q * k1]);
#pragma unroll
        for (int k1 = 0; k1 < L1; ++k1) lds[(q * L1 + k1) * PITCH + b] = x[k1];
      }
      __syncthreads();
      if (q < L1) {
#pragma unroll
        for (int n2 = 0; n2 < L2; ++n2) y[n2] = lds[(n2 * L1 + q) * PITCH + b];
        reg_fft<T, false, L2, kept_roots(L1 * L2)>(y);               // y[k2] = X[q + L1 k2]
      }
      if constexpr (MODE == ST_FWD) {
        if (pv[t] && q < L1) {
          auto store = [&](auto plain) {
#pragma unroll
            for (int k2 = 0; k2 < L2; ++k2) {
              const int kk = q + L1 * k2;
              if (kk < lout) {
                if constexpr (decltype(plain)::value) at_bytes(work, qb[t] + (unsigned)k2 * s1) = y[k2];
                else store_stream(&at_bytes(work, qb[t] + (unsigned)k2 * s1), y[k2]);
              }
            }
          };
          if (PLAIN == 1 || (PLAIN == 2 && p.plain_store)) store(std::true_type{});
          else store(std::false_type{});
        }
        continue;
      } else {
        if (pv[t] && q < L1) {
          // (v, r) = sum over the full spectrum of m |w^|^2 (Parseval), taken
          // as Re(conj(w^) m w^); this pencil's half-spectrum bin k_x stands for
          // itself and its mirror (weight gw)
          // (products of the bulk type, summed in FP64 like every inner product)
          double ws = 0.0;
#pragma unroll
          for (int k2 = 0; k2 < L2; ++k2) {
            const int kz = q + L1 * k2;
            T m = gm[t][k2];
            if (p.k0_from_slot && pen[t] == 0 && kz == 0) m = T(st->g0);
            const cplx<T> w = y[k2];
            y[k2] = cscale(w, m);
            ws += double(y[k2].x) * double(w.x) + double(y[k2].y) * double(w.y);
          }
          dacc += double(gw[t]) * ws;
        }
        __syncthreads();                        // step-2 reads of lds are done
      }
    } else {
      if (q < L1) {
#pragma unroll
        for (int k2 = 0; k2 < L2; ++k2) y[k2] = yin[t][k2];
      }
    }
    // inverse transform (ST_CONV second half, ST_INV)
    if (q < L1) {
      reg_fft<T, true, L2, kept_roots(L1 * L2)>(y);                  // y[n_a] = Z[q][n_a]
#pragma unroll
      for (int na = 1; na < L2; ++na) y[na] = cmul(y[na], cconj(tw[na * q]));
#pragma unroll
      for (int na = 0; na < L2; ++na) lds[(na * L1 + q) * PITCH + b] = y[na];
    }
    __syncthreads();
    if (q < L2) {
      cplx<T> x[L1];
#pragma unroll
      for (int k1 = 0; k1 < L1; ++k1) x[k1] = lds[(q * L1 + k1) * PITCH + b];
      reg_fft<T, true, L1, kept_roots(L1 * L2)>(x);                  // x[n_b] = out[q + L2 n_b]
      if (pv[t]) {
        auto store = [&](auto plain) {
#pragma unroll
          for (int nb = 0; nb < L1; ++nb) {
            const int e = q + L2 * nb;
            const bool out = PAD ? (nb < L1 / 2) : (e < lout);
            if (out) {
              if constexpr (decltype(plain)::value) at_bytes(work, qb[t] + (unsigned)nb * s2) = x[nb];
              else store_stream(&at_bytes(work, qb[t] + (unsigned)nb * s2), x[nb]);
            }
          }
        };
        if (MODE == ST_INV || PLAIN == 1 || (PLAIN == 2 && p.plain_store)) store(std::true_type{});
        else store(std::false_type{});
      }
    }
  }
  if constexpr (MODE == ST_CONV) {
    if (part_delta) {                           // one partial per wavefront
      const double sd = wave_sum(dacc);
      if ((tid & 63) == 0) part_delta[blockIdx.x * (NT / 64) + (tid >> 6)] = sd;
    }
  }
}

// ---------------------------------------------------------------------------
// x passes (pairs of real rows packed as one complex row)
// ---------------------------------------------------------------------------
// A work-group transforms 2P consecutive rows.  Row lengths are compile-time
// (PAD: the box holds L/2 points of the padded length L, else L), so every
// loop has a fixed trip count and all global loads of a thread are issued
// before the first one is used.
// P row pairs per work-group; the LDS pitch of a transform's elements is odd,
// so that the staging's stride of two elements per column spreads over the
// banks.
constexpr int xthreads(int L1, int L2, int P) { return round64(P * larger(L1, L2)); }

// Work-group sum for a compile-time block of NT threads: one wavefront needs
// no barrier.
template <int NT>
__device__ __forceinline__ double wg_sum(double v) {
  if constexpr (NT == 64) return wave_sum(v);
  else return block_sum(v);
}

// (row, column) of the element e = tid + i NT of a row-major tile with
// compile-time row length W, advanced in i without a division per element.
template <int W, int NT>
struct RowCol {
  int row, col;
  __device__ __forceinline__ explicit RowCol(int tid) : row(tid / W), col(tid - (tid / W) * W) {}
  __device__ __forceinline__ void next() {
    col += NT % W;
    row += NT / W;
    if (col >= W) {
      col -= W;
      ++row;
    }
  }
};

// Element idx of a buffer with a work-group-uniform base, addressed through a
// 32-bit byte offset (checked beside kMaxOffset).
#define GPS_AT(ptr, idx) at_bytes((ptr), (unsigned)(idx) * (unsigned)sizeof(*(ptr)))

// Work-buffer offsets of the NR consecutive rows row0, row0 + 1, ... of a
// tile (0 for rows past nrows).  row0 is work-group uniform, so the one division runs on the scalar
// unit and the offsets stay in scalar registers.
template <int NR, typename T>
__device__ __forceinline__ void tile_row_offsets(const XParams<T>& p, int row0, int Kx,
                                                 unsigned* off, bool* ok) {
  int pl = row0 / p.rows_per_plane;
  int rr = row0 - pl * p.rows_per_plane;
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    ok[j] = row0 + j < p.nrows;
    // rows past the end get offset 0, so that unconditional loads stay in bounds
    off[j] = ok[j] ? (unsigned)pl * (unsigned)p.plane_stride + (unsigned)rr * (unsigned)Kx : 0u;
    if (++rr == p.rows_per_plane) {
      rr = 0;
      ++pl;
    }
  }
}

// PLANE: the half spectrum goes to one plane per kx, half[kx][row] (the input
// of the plane pass): lanes run over the tile's rows, 2P consecutive values of
// every plane.
template <typename T, int L1, int L2, int P, int MODE, bool PAD, bool PLANE>
__global__ __launch_bounds__(xthreads(L1, L2, P))
void k_fxfwd(XParams<T> p) {
  constexpr bool SOLVE = MODE == XF_SOLVE || MODE == XF_SOLVE_REF;
  constexpr bool REF = MODE == XF_SOLVE_REF;     // also s += alpha sigma (refinement)
  constexpr int L = L1 * L2;
  constexpr int PITCH = P | 1;
  constexpr int NT = xthreads(L1, L2, P);
  constexpr int Lin = PAD ? L / 2 : L;
  constexpr int Kx = L / 2 + 1;
  constexpr int NIN = 2 * P * Lin;                 // real inputs of the tile
  constexpr int EIN = (NIN + NT - 1) / NT;
  constexpr int KI = (Kx + NT - 1) / NT;           // output bins per thread and row pair
  __shared__ cplx<T> lds[L * PITCH];
  __shared__ cplx<T> twl[L];
  T* ldsr = reinterpret_cast<T*>(lds);
  const int tid = threadIdx.x;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int row0 = tile * 2 * P;
  cplx<T>* work = p.work;
  const Slot<T> sl = p.tab.s[p.batch.slot[blockIdx.y]];
  if constexpr (SOLVE) work = sl.work;
  constexpr int ETW = (L + NT - 1) / NT;
  cplx<T> twv[ETW];
#pragma unroll
  for (int i = 0; i < ETW; ++i)
    twv[i] = load_parts(&p.tw[min(tid + i * NT, L - 1)]);   // clamped: no branch around the load
  // the head's own loads (state words, (p, Ap) partials) go first, then the
  // operands of the r update and of the transform (r, 1/sqrt(eps), Ap), then
  // those of the phi (and s) update (p, phi), which are used only after the
  // transform: the head waits only for its loads, the transform only for the
  // first group, and the second group arrives while the transform runs.
  // Operands are loaded even at k = 0 (unused there).
  XHead<NT == 64 ? 24 : 8> hd;                     // one (p, Ap) partial per x-inverse group
  if constexpr (SOLVE) xfwd_head_load(sl, p.n_pap_parts, hd);
  // rows are contiguous (row stride Lin, checked by the dispatcher), so
  // element e of the tile is at row0 * Lin + e
  const unsigned eo = (unsigned)row0 * (unsigned)Lin;
  const int nin = min(NIN, (p.nrows - row0) * Lin);     // tile elements that exist
  T rv[EIN], sv[EIN], pv[EIN], av[EIN];
  double fv[EIN];
  double gv[REF ? EIN : 1], cv[REF ? EIN : 1];   // sigma, s
  // Loads are unconditional: elements past the tile's end load its first
  // element (unused).  Without branches around the loads the compiler counts
  // them exactly and waits for each group alone.
#pragma unroll
  for (int i = 0; i < EIN; ++i) {
    const int e = tid + i * NT;
    const bool in = e < nin;
    const unsigned o = eo + (unsigned)(in ? e : 0);
    if constexpr (SOLVE) {
      const T r0 = GPS_AT(sl.r, o), s0 = GPS_AT(sl.isq, o);
      av[i] = GPS_AT(sl.ap, o);
      rv[i] = in ? r0 : T(0);
      sv[i] = in ? s0 : T(0);
    } else {
      const T r0 = T(GPS_AT(p.in_real, o));
      rv[i] = in ? r0 : T(0);
      sv[i] = T(0);
    }
  }
  if constexpr (SOLVE) {
#pragma unroll
    for (int i = 0; i < EIN; ++i) {
      const int e = tid + i * NT;
      const unsigned o = eo + (unsigned)(e < nin ? e : 0);
      pv[i] = GPS_AT(sl.p, o);
      fv[i] = GPS_AT(sl.phi, o);
      if constexpr (REF) {
        gv[i] = GPS_AT(sl.sig64, o);
        cv[i] = GPS_AT(sl.src64, o);
      }
    }
  }
  double alpha = 0.0;
  bool upd = false;
  if constexpr (SOLVE) {
    int k;
    if (!xfwd_head_finish(sl, p.n_pap_parts, hd, &k, &alpha, &upd)) return;
  }
  // phase 2: update, scale, stage the rows in LDS
  double mu = 0.0, rr = 0.0;
  // LDS float index of (row, x): 2 (x PITCH + row / 2) + row % 2 = 2 PITCH x + row
  RowCol<Lin, NT> rc(tid);
#pragma unroll
  for (int i = 0; i < EIN; ++i, rc.next()) {
    const int e = tid + i * NT;
    if (e < NIN) {
      T a = rv[i];
      if constexpr (SOLVE) {
        if (e < nin) {
          const unsigned o = eo + (unsigned)e;
          if (upd) {
            a = a - T(alpha) * av[i];
            GPS_AT(sl.r, o) = a;
          }
          rr += double(a) * double(a);
          a = a * sv[i];
          mu += double(a);
        }
      }
      ldsr[__umul24(2 * PITCH, (unsigned)rc.col) + rc.row] = a;
    }
  }
  if constexpr (PAD) {
#pragma unroll
    for (int i = 0; i < (P * (L - Lin) + NT - 1) / NT; ++i) {
      const int e = tid + i * NT;
      if (e < P * (L - Lin)) lds[(Lin + e / P) * PITCH + (e % P)] = cmk(T(0), T(0));
    }
  }
#pragma unroll
  for (int i = 0; i < ETW; ++i)
    if (tid + i * NT < L) twl[tid + i * NT] = cmk(twv[i].x, twv[i].y);
  __syncthreads();
  const int pp = tid % P;
  const int q = tid / P;
  const cplx<T>* tw = twl;
  cplx<T> x[L1];
  if (q < L2) {
#pragma unroll
    for (int n1 = 0; n1 < L1; ++n1) x[n1] = lds[(L2 * n1 + q) * PITCH + pp];
    reg_fft<T, false, L1, kept_roots(L1 * L2)>(x);
#pragma unroll
    for (int k1 = 1; k1 < L1; ++k1) x[k1] = cmul(x[k1], tw[q * k1]);
  }
  __syncthreads();
  if (q < L2) {
#pragma unroll
    for (int k1 = 0; k1 < L1; ++k1) lds[(q * L1 + k1) * PITCH + pp] = x[k1];
  }
  __syncthreads();
  cplx<T> y[L2];
  if (q < L1) {
#pragma unroll
    for (int n2 = 0; n2 < L2; ++n2) y[n2] = lds[(n2 * L1 + q) * PITCH + pp];
    reg_fft<T, false, L2, kept_roots(L1 * L2)>(y);
  }
  __syncthreads();
  if (q < L1) {
#pragma unroll
    for (int k2 = 0; k2 < L2; ++k2) lds[(q + L1 * k2) * PITCH + pp] = y[k2];
  }
  __syncthreads();
  if constexpr (PLANE) {
    constexpr int KS = NT / P;                      // threads that share a row pair
    cplx<T>* half = SOLVE ? sl.half : p.half;
    const int ra = row0 + 2 * pp;
    if (q < KS) {
#pragma unroll
      for (int i = 0; i < (Kx + KS - 1) / KS; ++i) {
        const int kk = q + i * KS;
        if (kk < Kx) {
          const cplx<T> zk = lds[kk * PITCH + pp];
          const cplx<T> zm = lds[(kk == 0 ? 0 : L - kk) * PITCH + pp];
          const T h = T(0.5);
          const unsigned o = (unsigned)kk * (unsigned)p.nrows + (unsigned)ra;
          if (ra < p.nrows) GPS_AT(half, o) = cmk(h * (zk.x + zm.x), h * (zk.y - zm.y));
          if (ra + 1 < p.nrows) GPS_AT(half, o + 1) = cmk(h * (zk.y + zm.y), h * (zm.x - zk.x));
        }
      }
    }
  } else {
    unsigned roff[2 * P];
    bool rok[2 * P];
    tile_row_offsets<2 * P>(p, row0, Kx, roff, rok);
#pragma unroll
    for (int p2 = 0; p2 < P; ++p2) {
#pragma unroll
      for (int i = 0; i < KI; ++i) {
        const int kk = tid + i * NT;
        if (kk < Kx) {
          const cplx<T> zk = lds[kk * PITCH + p2];
          const cplx<T> zm = lds[(kk == 0 ? 0 : L - kk) * PITCH + p2];
          const T half = T(0.5);
          if (rok[2 * p2])
            GPS_AT(work, roff[2 * p2] + kk) = cmk(half * (zk.x + zm.x), half * (zk.y - zm.y));
          if (rok[2 * p2 + 1])
            GPS_AT(work, roff[2 * p2 + 1] + kk) = cmk(half * (zk.y + zm.y), half * (zm.x - zk.x));
        }
      }
    }
  }
  if constexpr (SOLVE) {
    // phi += alpha p (and s += alpha sigma) of the previous iteration, after
    // the transform so that its operands' latency hides behind it
    if (upd) {
#pragma unroll
      for (int i = 0; i < EIN; ++i) {
        const int e = tid + i * NT;
        if (e < nin) {
          const unsigned o = eo + (unsigned)e;
          GPS_AT(sl.phi, o) = fv[i] + alpha * double(pv[i]);
          if constexpr (REF) GPS_AT(sl.src64, o) = cv[i] + alpha * gv[i];
        }
      }
    }
  }
  if constexpr (SOLVE) {                        // one partial per work-group
    const double s2 = wg_sum<NT>(rr);
    if (tid == 0) sl.part_rr[tile] = s2;
    if (p.periodic_mean) {
      const double s = wg_sum<NT>(mu);
      if (tid == 0) sl.part_mu[tile] = s;
    }
  }
}

// MODE XI_SOLVE / XI_SOLVE_PERIODIC / XI_SOLVE_REF: v = u / sqrt(eps) and the
// direction update of the PCG iteration (with the periodic mean term; with the
// refinement's sigma = r / sqrt(eps) + beta sigma); XI_REAL: plain output.
// PLANE: the rows are the sums of the plane pass's two parities,
//   row (z, y = j + m N) = work[kx][0][z][j] + (-1)^m work[kx][1][z][j],
// read with lanes over the tile's rows; in a solve an extra work-group (the
// first) takes the stop decision, and every work-group sums the plane pass's
// delta partials for beta (a few hundred values, one per plane and parity).
template <typename T, int L1, int L2, int P, int MODE, bool PAD, bool PLANE>
__global__ __launch_bounds__(xthreads(L1, L2, P))
void k_fxinv(XParams<T> p) {
  constexpr bool SOLVE = MODE != XI_REAL;
  constexpr bool PER = MODE == XI_SOLVE_PERIODIC;
  constexpr bool REF = MODE == XI_SOLVE_REF;
  constexpr int L = L1 * L2;
  constexpr int PITCH = P | 1;
  constexpr int NT = xthreads(L1, L2, P);
  constexpr int Lout = PAD ? L / 2 : L;
  constexpr int Kx = L / 2 + 1;
  constexpr int KI = (Kx + NT - 1) / NT;           // input bins per thread and row pair
  constexpr int NOUT = 2 * P * Lout;
  constexpr int EOUT = (NOUT + NT - 1) / NT;
  __shared__ cplx<T> lds[L * PITCH];
  __shared__ cplx<T> twl[L];
  const T* ldsr = reinterpret_cast<const T*>(lds);
  const int tid = threadIdx.x;
  constexpr int DEC = PLANE && SOLVE ? 1 : 0;      // the decision work-group
  const Slot<T> sl = p.tab.s[p.batch.slot[blockIdx.y]];
  if constexpr (DEC == 1) {
    if (blockIdx.x == 0) {
      pcg_decide(sl, p.dec);
      return;
    }
  }
  const int tile = xcd_tile(blockIdx.x, gridDim.x) - DEC;
  const int row0 = tile * 2 * P;
  cplx<T>* work = p.work;
  if constexpr (SOLVE) work = sl.work;
  // the y-inverse decision of this iteration (plain loads: written by an
  // earlier kernel, first used in the epilogue)
  DirArgs dir{};
  __shared__ int stopped;
  constexpr int NPS = NT == 64 ? 16 : 8;
  PartShare<DEC ? NPS : 4> sdl;
  PartShare<DEC && PER ? NPS : 4> smu;
  double dprev = 0.0;
  if constexpr (DEC == 1) {
    // (the decision work-group writes the other entry of delta only)
    const int k = sl.st->k;
    dir.fresh = k == 0;
    dprev = sl.st->delta[(k - 1) & 1];
    share_load(sdl, sl.part_delta, p.dec.n_delta);
    if constexpr (PER) share_load(smu, sl.part_mu, p.dec.n_rr);
  } else if constexpr (SOLVE) {
    dir.fresh = sl.st->fresh;
    dir.beta = sl.st->beta;
    dir.mu = PER ? sl.st->mu : 0.0;
  }
  constexpr int ETW = (L + NT - 1) / NT;
  cplx<T> twv[ETW];
#pragma unroll
  for (int i = 0; i < ETW; ++i)
    twv[i] = load_parts(&p.tw[min(tid + i * NT, L - 1)]);   // clamped: no branch around the load
  const int pp = tid % P;
  const int q = tid / P;
  constexpr int KS = NT / P;                       // PLANE: threads that share a row pair
  constexpr int KP = (Kx + KS - 1) / KS;
  cplx<T> xa[PLANE ? 1 : P][PLANE ? KP : KI], xb[PLANE ? 1 : P][PLANE ? KP : KI];
  if constexpr (PLANE) {
    cplx<T> ya[KP], yb[KP];
    const unsigned N = (unsigned)p.sh.N, pstride = (unsigned)p.sh.nz * N;
    unsigned off[2];
    bool ok[2], minus[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = row0 + 2 * pp + j;
      ok[j] = row < p.nrows;
      const unsigned rc = ok[j] ? (unsigned)row : 0u;   // rows past the end read row 0
      const unsigned z = fast_div(rc, p.sh.div_ny), y = rc - z * (unsigned)p.sh.ny;
      minus[j] = y >= N;
      off[j] = z * N + (minus[j] ? y - N : y);
    }
#pragma unroll
    for (int i = 0; i < KP; ++i) {
      const int kk = q + i * KS;
      const unsigned o = (unsigned)(kk < Kx ? kk : Kx - 1) * (2 * pstride);
      xa[0][i] = GPS_AT(work, o + off[0]);
      xb[0][i] = GPS_AT(work, o + off[1]);
      ya[i] = GPS_AT(work, o + pstride + off[0]);
      yb[i] = GPS_AT(work, o + pstride + off[1]);
    }
#pragma unroll
    for (int i = 0; i < KP; ++i) {
      xa[0][i] = minus[0] ? csub(xa[0][i], ya[i]) : cadd(xa[0][i], ya[i]);
      xb[0][i] = minus[1] ? csub(xb[0][i], yb[i]) : cadd(xb[0][i], yb[i]);
    }
#pragma unroll
    for (int i = 0; i < KP; ++i) {
      if (!ok[0]) xa[0][i] = cmk(T(0), T(0));
      if (!ok[1]) xb[0][i] = cmk(T(0), T(0));
    }
  } else {
    unsigned roff[2 * P];
    bool rok[2 * P];
    tile_row_offsets<2 * P>(p, row0, Kx, roff, rok);
#pragma unroll
    for (int p2 = 0; p2 < P; ++p2) {
#pragma unroll
      for (int i = 0; i < KI; ++i) {
        const int kk = tid + i * NT;
        const int kc = kk < Kx ? kk : Kx - 1;        // clamped: branch-free loads
        const cplx<T> va = GPS_AT(work, roff[2 * p2] + kc);
        const cplx<T> vb = GPS_AT(work, roff[2 * p2 + 1] + kc);
        xa[p2][i] = rok[2 * p2] ? va : cmk(T(0), T(0));
        xb[p2][i] = rok[2 * p2 + 1] ? vb : cmk(T(0), T(0));
      }
    }
  }
  // the stop flag right after the rows: the transform waits for both, and the
  // epilogue operands below stay in flight while it runs
  int stop = 0;
  if constexpr (SOLVE) stop = stop_flag_issue(sl.st);
  // epilogue operands are independent of the transform: load them now too
  constexpr int EO = SOLVE ? EOUT : 1;
  T sv[EO], rv[EO], qv[EO], pv[EO], av[EO], mv[PER ? EOUT : 1];
  double gv[REF ? EOUT : 1];                     // sigma
  // rows are contiguous (row stride Lout, checked by the dispatcher)
  const unsigned eo = (unsigned)row0 * (unsigned)Lout;
  const int nout = min(NOUT, (p.nrows - row0) * Lout);  // tile elements that exist
  if constexpr (SOLVE) {
    // unconditional loads (elements past the tile's end load its first
    // element, unused): no branches, so the transform waits for the row loads
    // alone
#pragma unroll
    for (int i = 0; i < EOUT; ++i) {
      const int e = tid + i * NT;
      const unsigned o = eo + (unsigned)(e < nout ? e : 0);
      sv[i] = GPS_AT(sl.isq, o);
      rv[i] = GPS_AT(sl.r, o);
      qv[i] = GPS_AT(sl.qk, o);
      pv[i] = GPS_AT(sl.p, o);
      av[i] = GPS_AT(sl.ap, o);
      if constexpr (PER) mv[i] = GPS_AT(sl.s, o);
      if constexpr (REF) gv[i] = GPS_AT(sl.sig64, o);
    }
    if constexpr (DEC == 0) {
      if (stop_flag_set(stop)) return;
    } else {
      // the decision work-group may set the flag during this launch: one thread's
      // copy, read after the staging's barrier, holds for the whole work-group
      if (tid == 0) stopped = stop;
    }
  }
#pragma unroll
  for (int p2 = 0; p2 < (PLANE ? 1 : P); ++p2)
#pragma unroll
  for (int i = 0; i < (PLANE ? KP : KI); ++i) {
    const int kk = PLANE ? q + i * KS : tid + i * NT;
    const int pr = PLANE ? pp : p2;                // row pair of the tile
    if (kk < Kx && (!PLANE || q < KS)) {
      cplx<T> a = xa[p2][i], b = xb[p2][i];
      if (kk == 0 || 2 * kk == L) {    // self-conjugate bins of a real row
        a.y = T(0);
        b.y = T(0);
      }
      lds[kk * PITCH + pr] = cmk(a.x - b.y, a.y + b.x);
      const int km = L - kk;
      if (kk > 0 && km >= Kx) lds[km * PITCH + pr] = cmk(a.x + b.y, b.x - a.y);
    }
  }
#pragma unroll
  for (int i = 0; i < ETW; ++i)
    if (tid + i * NT < L) twl[tid + i * NT] = cmk(twv[i].x, twv[i].y);
  __syncthreads();
  if constexpr (DEC == 1) {
    if (stopped) return;
  }
  const cplx<T>* tw = twl;
  cplx<T> y[L2];
  if (q < L1) {
#pragma unroll
    for (int k2 = 0; k2 < L2; ++k2) y[k2] = lds[(q + L1 * k2) * PITCH + pp];
    reg_fft<T, true, L2, kept_roots(L1 * L2)>(y);
#pragma unroll
    for (int na = 1; na < L2; ++na) y[na] = cmul(y[na], cconj(tw[na * q]));
  }
  __syncthreads();
  if (q < L1) {
#pragma unroll
    for (int na = 0; na < L2; ++na) lds[(na * L1 + q) * PITCH + pp] = y[na];
  }
  __syncthreads();
  cplx<T> x[L1];
  if (q < L2) {
#pragma unroll
    for (int k1 = 0; k1 < L1; ++k1) x[k1] = lds[(q * L1 + k1) * PITCH + pp];
    reg_fft<T, true, L1, kept_roots(L1 * L2)>(x);
  }
  __syncthreads();
  if (q < L2) {
#pragma unroll
    for (int nb = 0; nb < L1; ++nb) lds[(q + L2 * nb) * PITCH + pp] = x[nb];
  }
  __syncthreads();
  if constexpr (DEC == 1) {
    const double delta = share_sum(sdl, sl.part_delta, p.dec.n_delta);
    dir.beta = dir.fresh ? 0.0 : delta / dprev;
    if constexpr (PER) dir.mu = share_sum(smu, sl.part_mu, p.dec.n_rr) / p.dec.npts;
  }
  if constexpr (SOLVE) {
    double acc = 0.0;
    RowCol<Lout, NT> rc(tid);
#pragma unroll
    for (int i = 0; i < EOUT; ++i, rc.next()) {
      const int e = tid + i * NT;
      if (e < nout) {
        const unsigned o = eo + (unsigned)e;
        const T v = ldsr[__umul24(2 * PITCH, (unsigned)rc.col) + rc.row] * sv[i];
        T pn = pv[i], an = av[i];
        if constexpr (REF) {
          const double w = double(rv[i] * sv[i]);   // the preconditioner input of this iteration
          GPS_AT(sl.sig64, o) = dir.fresh ? w : w + dir.beta * gv[i];
        }
        direction_update(v, rv[i], qv[i], PER ? mv[i] : T(0), pn, an, dir);
        GPS_AT(sl.p, o) = pn;
        GPS_AT(sl.ap, o) = an;
        acc += double(pn) * double(an);
      }
    }
    const double s1 = wg_sum<NT>(acc);          // one partial per work-group
    if (tid == 0) sl.part_pap[tile] = s1;
  } else {
    RowCol<Lout, NT> rc(tid);
#pragma unroll
    for (int i = 0; i < EOUT; ++i, rc.next()) {
      const int e = tid + i * NT;
      if (e < nout) GPS_AT(p.out_real, eo + (unsigned)e) = double(ldsr[__umul24(2 * PITCH, (unsigned)rc.col) + rc.row]);
    }
  }
}

// ---------------------------------------------------------------------------
// launches of one length
// ---------------------------------------------------------------------------
// Tiles per work-group of the strided passes.
constexpr int kStridedTiles = 1;

// L = L1 L2; P row pairs per work-group of the x passes.  Strided passes of
// the tuned lengths choose the store kind at compile time (a branch in the
// store loop cost 0.75 us in the 96^3 y forward); the others branch on
// SParams::plain_store once, around two store loops.
template <int L1, int L2, int P, bool TUNED> struct TwoLevel {
  static constexpr int L = L1 * L2;

  template <typename T, int MODE, bool PAD, int B>
  static void strided_b(const SParams<T>& p, dim3 grid, hipStream_t s) {
    const dim3 blk(round64(B * larger(L1, L2)));
    if constexpr (MODE == ST_INV) {
      GPS_LAUNCH((k_fstrided<T, L1, L2, MODE, PAD, kStridedTiles, B, 0>), grid, blk, 0, s, p);
    } else if constexpr (TUNED) {
      if (p.plain_store)
        GPS_LAUNCH((k_fstrided<T, L1, L2, MODE, PAD, kStridedTiles, B, 1>), grid, blk, 0, s, p);
      else
        GPS_LAUNCH((k_fstrided<T, L1, L2, MODE, PAD, kStridedTiles, B, 0>), grid, blk, 0, s, p);
    } else {
      GPS_LAUNCH((k_fstrided<T, L1, L2, MODE, PAD, kStridedTiles, B, 2>), grid, blk, 0, s, p);
    }
  }

  template <typename T, bool PAD>
  static void strided_p(int mode, const SParams<T>& p, hipStream_t s) {
    constexpr int B = strided_tile<T>(L);
    const int dec = mode == ST_INV && (p.decide || p.sc.st) ? 1 : 0;   // the decision work-group
    constexpr int W = B * kStridedTiles;
    const dim3 grid((p.npencils + W - 1) / W + dec, p.work ? 1 : p.batch.n);
    if (mode == ST_FWD) strided_b<T, ST_FWD, PAD, B>(p, grid, s);
    else if (mode == ST_INV) strided_b<T, ST_INV, PAD, B>(p, grid, s);
    else strided_b<T, ST_CONV, PAD, B>(p, grid, s);
  }

  template <typename T> static void strided(int mode, const SParams<T>& p, hipStream_t s) {
    // PAD when the pencil's data half is L/2: forward reads, z pass reads and
    // writes, inverse writes that half only
    if constexpr (L1 % 2 == 0) {
      if ((mode == ST_FWD && 2 * p.Lin == L) ||
          (mode == ST_CONV && 2 * p.Lin == L && p.Lout == p.Lin) ||
          (mode == ST_INV && 2 * p.Lout == L && p.Lin == L)) {
        strided_p<T, true>(mode, p, s);
        return;
      }
    }
    strided_p<T, false>(mode, p, s);
  }

  // The x passes exist for full rows (PAD = false) and for half-padded rows
  // (PAD: L/2 points), the periodic mean term on full rows only (a padded x
  // axis is not periodic); beside the plane pass there is no refinement
  // and no FP64 solve (beside_plane).
  template <typename T, bool PAD>
  static void xfwd_p(int mode, const XParams<T>& p, dim3 grid, hipStream_t s) {
    const dim3 blk(xthreads(L1, L2, P));
    if constexpr (L <= kPlaneMaxLx) {
      if (p.sh.N > 0) {
        if constexpr (sizeof(T) == sizeof(float)) {
          if (mode == XF_SOLVE) {
            GPS_LAUNCH((k_fxfwd<T, L1, L2, P, XF_SOLVE, PAD, true>), grid, blk, 0, s, p);
            return;
          }
        }
        GPS_LAUNCH((k_fxfwd<T, L1, L2, P, XF_REAL, PAD, true>), grid, blk, 0, s, p);
        return;
      }
    }
    if (mode == XF_SOLVE && p.refine) {
      if constexpr (six_fit<T, PAD>())
        GPS_LAUNCH((k_fxfwd<T, L1, L2, P, XF_SOLVE_REF, PAD, false>), grid, blk, 0, s, p);
    } else if (mode == XF_SOLVE) {
      GPS_LAUNCH((k_fxfwd<T, L1, L2, P, XF_SOLVE, PAD, false>), grid, blk, 0, s, p);
    } else {
      GPS_LAUNCH((k_fxfwd<T, L1, L2, P, XF_REAL, PAD, false>), grid, blk, 0, s, p);
    }
  }
  template <typename T, bool PAD, bool PLANE>
  static void xinv_m(int mode, const XParams<T>& p, dim3 grid, hipStream_t s) {
    const dim3 blk(xthreads(L1, L2, P));
    if constexpr (PLANE && sizeof(T) != sizeof(float)) {
      GPS_LAUNCH((k_fxinv<T, L1, L2, P, XI_REAL, PAD, PLANE>), grid, blk, 0, s, p);
      return;
    }
    if constexpr (!PAD && six_fit<T, PAD>()) {
      if (mode == XI_SOLVE && p.periodic_mean) {
        GPS_LAUNCH((k_fxinv<T, L1, L2, P, XI_SOLVE_PERIODIC, PAD, PLANE>), grid, blk, 0, s, p);
        return;
      }
    }
    if constexpr (!PLANE && six_fit<T, PAD>()) {
      if (mode == XI_SOLVE && p.refine) {
        GPS_LAUNCH((k_fxinv<T, L1, L2, P, XI_SOLVE_REF, PAD, PLANE>), grid, blk, 0, s, p);
        return;
      }
    }
    if (mode == XI_SOLVE)
      GPS_LAUNCH((k_fxinv<T, L1, L2, P, XI_SOLVE, PAD, PLANE>), grid, blk, 0, s, p);
    else
      GPS_LAUNCH((k_fxinv<T, L1, L2, P, XI_REAL, PAD, PLANE>), grid, blk, 0, s, p);
  }
  template <typename T, bool PAD>
  static void xinv_p(int mode, const XParams<T>& p, dim3 grid, hipStream_t s) {
    if constexpr (L <= kPlaneMaxLx) {
      if (p.sh.N > 0) {
        if (mode == XI_SOLVE) grid.x += 1;             // the decision work-group
        xinv_m<T, PAD, true>(mode, p, grid, s);
        return;
      }
    }
    xinv_m<T, PAD, false>(mode, p, grid, s);
  }

  template <typename T> static dim3 xgrid(const XParams<T>& p) {
    return dim3(((p.nrows + 1) / 2 + P - 1) / P, p.has_slots ? p.batch.n : 1);
  }

  // A thread of the solve's x inverse holds 4 P KI values of the rows and its points'
  // fields.  FP64 solves with six fields on full rows of 324, 378, 400, 420 and 432 points (544 to
  // 576 registers, 528 at 378) spill 44 to 126 of 512, and were slower than the generic passes:
  // periodic 0.90 to 0.97 x (378: 0.996), refined 0.85 to 0.98.  At up to 504 (360: 40 spilled)
  // the two-level ones win: 1.05 to 1.2.
  template <typename T, bool PAD> static constexpr bool six_fit() {
    constexpr int NT = xthreads(L1, L2, P), Lout = PAD ? L / 2 : L;
    constexpr int KI = (L / 2 + 1 + NT - 1) / NT, EOUT = (2 * P * Lout + NT - 1) / NT;
    return int(sizeof(T) / 4) * (4 * P * KI + 6 * EOUT) < 528;
  }
  template <typename T> static bool six_fields(const XParams<T>& p) {
    return p.refine || p.periodic_mean;
  }

  template <typename T> static bool beside_plane(bool solve, const XParams<T>& p) {
    return L <= kPlaneMaxLx && (!solve || (sizeof(T) == sizeof(float) && !p.refine));
  }

  template <typename T> static bool xfwd(int mode, const XParams<T>& p, hipStream_t s) {
    if (mode != XF_SOLVE && mode != XF_REAL) return false;
    if (p.sh.N > 0 && !beside_plane(mode == XF_SOLVE, p)) return false;
    if (p.in_row_stride != p.Lin) return false;        // the kernels assume contiguous rows
    if (p.Lin == L) {
      if (mode == XF_SOLVE && six_fields(p) && !six_fit<T, false>()) return false;
      xfwd_p<T, false>(mode, p, xgrid(p), s);
      return true;
    }
    if constexpr (L1 % 2 == 0) {
      if (2 * p.Lin == L) {
        xfwd_p<T, true>(mode, p, xgrid(p), s);
        return true;
      }
    }
    return false;
  }

  template <typename T> static bool xinv(int mode, const XParams<T>& p, hipStream_t s) {
    if (p.sh.N > 0 && !beside_plane(mode == XI_SOLVE, p)) return false;
    if (p.in_row_stride != p.Lout) return false;       // the kernels assume contiguous rows
    if (p.Lout == L) {
      if (mode == XI_SOLVE && six_fields(p) && !six_fit<T, false>()) return false;
      xinv_p<T, false>(mode, p, xgrid(p), s);
      return true;
    }
    if constexpr (L1 % 2 == 0) {
      if (2 * p.Lout == L) {
        xinv_p<T, true>(mode, p, xgrid(p), s);
        return true;
      }
    }
    return false;
  }

  // The FP32 x passes alone (grids of few rows).
  static LengthPasses x_passes32() {
    return LengthPasses{L, L1, L2, P, false, nullptr, nullptr, &TwoLevel::template xfwd<float>, nullptr,
                        &TwoLevel::template xinv<float>, nullptr};
  }

  static LengthPasses passes() {
    return LengthPasses{L, L1, L2, P, six_fit<double, false>(),
                        &TwoLevel::template strided<float>, &TwoLevel::template strided<double>,
                        &TwoLevel::template xfwd<float>, &TwoLevel::template xfwd<double>,
                        &TwoLevel::template xinv<float>, &TwoLevel::template xinv<double>};
  }
};

}  // namespace gps
