// Stop decision of Algorithm SC and the PSD minimization (device side).
#pragma once

#include "gps.h"
#include "gps_device.h"
#include "gps_launch.h"

namespace gps {

// ---------------------------------------------------------------------------
// Stop decision of an SC/PSD step (one work-group): from the update's partial
// pairs (||r||^2, ||r/eps||^2) it records the step, its norms and the status,
// and sets done on convergence, failure or the step limit.  It acts only when
// the update has marked a decision pending, so every update is decided once,
// whether by the next step's y-inverse pass or by a launch of its own.
// ---------------------------------------------------------------------------
__device__ inline void sc_decide_group(const double* __restrict__ part, int nparts, ScState* st) {
  if (st->done || !st->pending) return;          // the same for every thread
  const double rr = sum_partials(part, nparts, 2);
  const double ff = sum_partials(part + 1, nparts, 2);
  if (threadIdx.x != 0) return;
  ScState z = *st;
  z.pending = 0;
  if (z.status != GPS_E_NOT_CONVERGED) {          // breakdown or non-finite step
    z.done = 1;
    *st = z;
    return;
  }
  const int step = z.step;
  z.ff_prev = z.ff;
  z.rr = rr;
  z.ff = ff;
  z.step = step + 1;
  if (!isfinite(rr) || !isfinite(ff)) {
    z.status = GPS_E_NONFINITE;
  } else if (z.method == GPS_METHOD_SC) {
    // SC's residual ||rho_iter_{k+1} - rho_iter_k|| = (eta/4 pi) ||r_k/eps|| of
    // the iterate before this step; the first step is the unmixed phi_0
    if (step >= 1) {
      z.iters = step;
      if (z.eta / kFourPi * sqrt(z.ff_prev) <= z.thr_sc) z.status = GPS_OK;
    }
  } else {
    z.iters = step + 1;
    if (z.method == GPS_METHOD_PSD ? sqrt(rr) <= z.thr_r : sqrt(ff) <= z.thr_w) z.status = GPS_OK;
  }
  if (z.status != GPS_E_NOT_CONVERGED || z.step >= z.max_steps) z.done = 1;
  *st = z;
}

}  // namespace gps
