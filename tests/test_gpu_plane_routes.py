"""Plans whose vacuum solves take the plane pass while their PCG solves keep the y, z and y
passes (FP64, and FP32 on large grids), the calls in turn on one plan: the half spectrum that
the first vacuum solve adds leaves the solves' bits alone.  Tolerances of the parity tests."""
import numpy as np
import pytest

import plane_rule
from oracle import green, pcg
from paper_1509_00680_amd import gps
from gpu_util import dev, host, empty, plan, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,bc,precision", [((60, 160, 168), "periodic", "mixed"),
                                                ((24, 20, 18), "free", "fp64")])
def test_solves_and_vacuum_solves_in_turn(shape, bc, precision):
    require_gpu()
    elem = 4 if precision == "mixed" else 8
    assert plane_rule.plane(shape, bc, elem) == (True, False)
    rng = np.random.default_rng(23)
    z, y, x = np.meshgrid(*[2.0 * np.pi * np.arange(m) / m for m in shape], indexing="ij")
    eps = 6.0 + 2.0 * np.cos(x) * np.cos(y) + np.sin(z)
    rho = rng.normal(size=shape)
    rho -= rho.mean()
    expect = green.VacuumSolver(shape, 0.45, bc).apply(rho)
    p = plan(shape, 0.45, bc, precision)
    d_rho, d_eps = dev(rho), dev(eps)
    phi, u = empty(shape), empty(shape)
    tol = 1e-6 if precision == "mixed" else 1e-10
    first, held = None, None
    for turn in range(2):
        print("plane routes", shape, bc, precision, turn, flush=True)
        assert p.solve_generalized(d_rho, d_eps, phi, tol) == gps.GPS_OK
        if first is None:
            first, held = host(phi), p.device_bytes()
        assert np.array_equal(host(phi), first)
        assert p.solve_vacuum(d_rho, u) == gps.GPS_OK
        half = shape[0] * shape[1] * (plane_rule.lengths(shape, bc)[0] // 2 + 1) * 2 * elem
        assert p.device_bytes() == held + half
        assert np.abs(host(u) - expect).max() <= (3e-6 if elem == 4 else 1e-12) * \
            np.abs(expect).max()
    ref = pcg.pcg_solve(rho, eps, 0.45, bc, tol=1e-9)
    lam = eps.min() * (2.0 * np.pi / (0.45 * max(shape))) ** 2
    assert np.linalg.norm(first - ref.phi) <= 2.0 * tol * 4.0 * np.pi * np.linalg.norm(rho) / lam
    p.close()
