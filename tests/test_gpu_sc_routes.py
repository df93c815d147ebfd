"""Algorithm SC and the PSD steps on grids whose y inverse, which also takes the stop
decisions, runs in the generic passes (length 12) and in the two-level ones (30), after odd and
even numbers of steps, the methods one after the other on one plan.  FP64, against the oracle's
iterates within 1e-10 of max|phi| (the tolerance of the SC parity tests)."""
import numpy as np
import pytest

from oracle import sc
from paper_1509_00680_amd import gps
from gpu_util import dev, host, empty, plan, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(18, 6, 10), (9, 15, 16)])
@pytest.mark.parametrize("steps", [1, 2, 7])
def test_iterates_on_both_y_passes(shape, steps):
    require_gpu()
    rng = np.random.default_rng(41)
    z, y, x = np.meshgrid(*[np.linspace(-1.0, 1.0, n) for n in shape], indexing="ij")
    rho = rng.normal(size=shape)
    eps = 1.0 + 30.0 / (1.0 + np.exp(-6.0 * (z * z + y * y + x * x - 0.6)))
    pl = plan(shape, 0.5, "free", "fp64", maxit=steps)
    phi = empty(shape)
    for method in ("sc", "psd", "psd_weighted", "sc"):
        if method == "sc":
            ref, _, _ = sc.sc_solve(rho, eps, 0.5, "free", 0.6, tol=0.0, maxit=steps)
        else:
            ref, _, _ = sc.psd_solve(rho, eps, 0.5, "free", tol=0.0, maxit=steps,
                                     step="paper" if method == "psd" else "weighted")
        print("sc routes", shape, steps, method, flush=True)
        st = pl.solve_sc(dev(rho), dev(eps), phi, 1e-30, method=method, eta=0.6)
        assert st == gps.GPS_E_NOT_CONVERGED, gps.STATUS[st]
        assert pl.info()["iterations"] == steps
        assert np.abs(host(phi) - ref).max() <= 1e-10 * np.abs(ref).max()
