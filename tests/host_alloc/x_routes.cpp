// Prints, for every x length of full rows, which x passes PCG solves launch: one line per
// length, boundary condition, precision and refinement.
#include <cstdio>
#include <vector>

#include "fake_hip.h"
#include "gps.h"

static bool smooth(int n) {
  for (int f : {2, 3, 5, 7})
    while (n % f == 0) n /= f;
  return n == 1;
}

int main() {
  for (int nx = 8; nx <= 512; ++nx) {
    if (!smooth(nx)) continue;
    const std::vector<double> rho((size_t)nx * 16, 0.0), eps(rho.size(), 1.0);
    std::vector<double> phi(rho.size());
    for (int bc : {GPS_BC_SURFACE, GPS_BC_PERIODIC})
      for (int precision : {GPS_PREC_FP64, GPS_PREC_MIXED})
        for (int refine : {0, 5}) {
          if (refine && bc == GPS_BC_PERIODIC) continue;
          gps_plan* p = nullptr;
          if (gps_plan_create(nx, 4, 4, 0.5, bc, &p) != GPS_OK) return 1;
          gps_options o;
          gps_plan_get_options(p, &o);
          o.precision = precision;
          o.refine_every = refine;
          if (gps_plan_set_options(p, &o) != GPS_OK) return 1;
          fake::launches.clear();
          if (gps_solve_generalized(p, rho.data(), eps.data(), phi.data(), 1e-6) != GPS_OK) return 1;
          // (both passes of a solve: their partial sums are counted alike)
          const char* type = precision == GPS_PREC_FP64 ? "Id" : "If";
          int n[4] = {};
          for (const auto& l : fake::launches) {
            const std::string& k = l.first;
            if (k.find(type) == std::string::npos) continue;
            // XF_SOLVE, XI_SOLVE and their forms; not the plain transforms of a refinement
            const bool plain = k.find("ELi1ELb") != std::string::npos ||
                               k.find("Li1EE") != std::string::npos;
            if (plain) continue;
            if (k.find("k_fxfwd") != std::string::npos) n[0] += l.second;
            else if (k.find("k_fxinv") != std::string::npos) n[1] += l.second;
            else if (k.find("k_xfwd") != std::string::npos) n[2] += l.second;
            else if (k.find("k_xinv") != std::string::npos) n[3] += l.second;
          }
          const bool fast = n[0] > 0 && n[0] == n[1] && n[2] == 0 && n[3] == 0;
          const bool generic = n[2] > 0 && n[2] == n[3] && n[0] == 0 && n[1] == 0;
          std::printf("%d %s %s %d %s\n", nx, bc == GPS_BC_PERIODIC ? "periodic" : "surface",
                      precision == GPS_PREC_FP64 ? "fp64" : "mixed", refine,
                      fast ? "two-level" : generic ? "generic" : "mixed-up");
          gps_plan_destroy(p);
        }
  }
  return 0;
}
