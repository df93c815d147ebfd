// The x passes beside the plane pass (XParams::sh.N > 0) exist for plain transforms and for
// the FP32 solve without refinement.  Any other mode is refused before a launch, never run as
// another one; so are lengths without such passes.  Exit status 0 = pass.
#include <cstdio>

#include "fake_hip.h"
#include "gps_launch.h"

static int failures = 0, checks = 0;
static void expect(bool ok, const char* what, int elem, int mode, int refine, int L) {
  ++checks;
  if (ok) return;
  ++failures;
  std::fprintf(stderr, "FAILED %s: %s, mode %d, refine %d, length %d\n", what,
               elem == 4 ? "FP32" : "FP64", mode, refine, L);
}

template <typename T, typename F>
static void try_mode(F launch, const char* kernel, int mode, int solve, int refine, int L) {
  gps::XParams<T> p{};
  p.g.nx = p.Lin = p.Lout = L;
  p.g.Lx = L;
  p.nrows = 8;
  p.rows_per_plane = 4;
  p.in_row_stride = L;
  p.P = 1;
  p.batch.n = 1;
  p.refine = refine;
  p.sh.N = 2;
  const bool exists = L == 32 && (mode != solve || (sizeof(T) == sizeof(float) && !refine));
  fake::launches.clear();
  bool refused = false;
  try {
    launch(mode, p, nullptr);
  } catch (const gps::DevError&) {
    refused = true;
  }
  expect(refused == !exists, "refused", sizeof(T), mode, refine, L);
  expect(fake::count("") == exists && fake::count(kernel) == exists, "launches", sizeof(T), mode,
         refine, L);
}

template <typename T> static void all() {
  for (int L : {32, 8, 256, 1024})
    for (int refine : {0, 1}) {
      for (int mode : {gps::XF_REAL, gps::XF_SOLVE})
        try_mode<T>(gps::launch_xfwd<T>, "k_fxfwd", mode, gps::XF_SOLVE, mode == gps::XF_SOLVE && refine, L);
      for (int mode : {gps::XI_REAL, gps::XI_SOLVE})
        try_mode<T>(gps::launch_xinv<T>, "k_fxinv", mode, gps::XI_SOLVE, mode == gps::XI_SOLVE && refine, L);
    }
}

// The plane kernel reads a solve's slot in FP32 alone.
template <typename T> static void slots() {
  gps::Geom g{};
  g.nx = g.ny = g.nz = 16;
  g.Lx = g.Ly = g.Lz = 32;
  g.Kx = 17;
  gps::PlaneParams<T> p{};
  p.sh = gps::plane_shape(g, sizeof(T));
  p.Kx = g.Kx;
  p.batch.n = 1;
  gps::cplx<T> buffer{};
  for (gps::cplx<T>* work : {static_cast<gps::cplx<T>*>(nullptr), &buffer}) {
    p.work = work;
    fake::launches.clear();
    bool refused = false;
    try {
      gps::launch_plane<T>(p, nullptr);
    } catch (const gps::DevError&) {
      refused = true;
    }
    expect(refused == (!work && sizeof(T) == sizeof(double)), "slots", sizeof(T), 0, 0, 32);
    expect(fake::count("k_plane") == !refused, "slot launches", sizeof(T), 0, 0, 32);
  }
}

int main() {
  all<float>();
  all<double>();
  slots<float>();
  slots<double>();
  std::printf("plane modes: %d checks, %d failures\n", checks, failures);
  return failures == 0 ? 0 : 1;
}
