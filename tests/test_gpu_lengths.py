"""GPU parity of every two-level FFT length against the FP64 oracle: the length on each
axis of the vacuum solver, padded (isolated axis) and full (periodic axis), and as the x axis
of generalized Poisson solves.  Tolerances are those of the other parity tests: 1e-12 (FP64)
and 3e-6 (mixed) of max|u| for one vacuum solve; 1e-8 of max|phi| (FP64) and 1e-5 (mixed,
isolated axes) for a solve.  The periodic cells here are up to 90 times longer than wide, where
a relative residual tol leaves an error of up to tol ||b|| / lambda, lambda = min(eps) (2 pi /
length)^2 the smallest eigenvalue; the mixed solves there are held to twice that norm (the FP32
recursion's residual drifts from the true one)."""
import numpy as np
import pytest

from oracle import green, pcg
from paper_1509_00680_amd import gps
from gpu_util import dev, host, empty, plan, require_gpu
from test_fft_lengths import SPLITS

pytestmark = pytest.mark.gpu


def _cases(L):
    return [("free", L // 2), ("periodic", L)] if L % 2 == 0 else [("periodic", L)]


@pytest.mark.parametrize("L", sorted(SPLITS))
def test_vacuum_every_axis(L):
    require_gpu()
    rng = np.random.default_rng(L)
    for bc, n in _cases(L):
        # nz = 2 keeps the y, z, y passes beside the x length, 5 takes the plane pass up to 200
        for shape in ((5, 3, n), (2, 3, n), (3, n, 5), (n, 5, 3)):
            f = rng.normal(size=shape)
            if bc == "periodic":
                f -= f.mean()
            expect = green.VacuumSolver(shape, 0.45, bc).apply(f)
            for precision, tol in (("fp64", 1e-12), ("mixed", 3e-6)):
                print("vacuum length", L, bc, shape, precision, flush=True)
                p = plan(shape, 0.45, bc, precision)
                u = empty(shape)
                assert p.solve_vacuum(dev(f), u) == gps.GPS_OK
                assert np.abs(host(u) - expect).max() <= tol * np.abs(expect).max()
                p.close()


@pytest.mark.parametrize("L", sorted(SPLITS))
def test_solve_along_x(L):
    require_gpu()
    rng = np.random.default_rng(1000 + L)
    # nz = 2 keeps the y, z, y passes beside an x length that may have the plane pass (up to 200;
    # beyond, both depths take them, and FP32 PCG breaks down on some 2 x 5 x 300 cells)
    for bc, n, nz in [(bc, n, nz) for bc, n in _cases(L) for nz in ((6, 2) if L <= 200 else (6,))]:
        shape = (nz, 5, n)
        z, y, x = np.meshgrid(*[2.0 * np.pi * np.arange(m) / m for m in shape], indexing="ij")
        eps = 6.0 + 2.0 * np.cos(x) * np.cos(y) + np.sin(z)
        rho = rng.normal(size=shape)
        if bc == "periodic":
            rho -= rho.mean()
        ref = pcg.pcg_solve(rho, eps, 0.5, bc, tol=1e-11)
        for precision, tol in (("fp64", 1e-11), ("mixed", 1e-6)):
            print("solve length", L, bc, shape, precision, flush=True)
            p = plan(shape, 0.5, bc, precision)
            phi = empty(shape)
            assert p.solve_generalized(dev(rho), dev(eps), phi, tol) == gps.GPS_OK
            err = host(phi) - ref.phi
            if precision == "mixed" and bc == "periodic":
                lam = eps.min() * (2.0 * np.pi / (0.5 * n)) ** 2
                assert np.linalg.norm(err) <= 2.0 * tol * 4.0 * np.pi * np.linalg.norm(rho) / lam
            else:
                bound = 1e-8 if precision == "fp64" else 1e-5
                assert np.abs(err).max() <= bound * np.abs(ref.phi).max()
            p.close()


@pytest.mark.parametrize("ny,nz", [(63, 63), (64, 64), (49, 84), (63, 75)])
@pytest.mark.parametrize("n", [32, 48, 64])
def test_row_pairs_by_row_count(n, ny, nz):
    """Lengths 32, 48 and 64 take fewer row pairs per work-group up to 4096 rows: grids on both
    sides of that line and on it, with full and partly filled last work-groups."""
    require_gpu()
    rng = np.random.default_rng(n)
    shape, h = (nz, ny, n), 0.45
    z, y, x = np.meshgrid(*[2.0 * np.pi * np.arange(m) / m for m in shape], indexing="ij")
    eps = 6.0 + 2.0 * np.cos(x) * np.cos(y) + np.sin(z)
    f = rng.normal(size=shape)
    f -= f.mean()
    expect = green.VacuumSolver(shape, h, "periodic").apply(f)
    ref = pcg.pcg_solve(f, eps, h, "periodic", tol=1e-11)
    lam = eps.min() * (2.0 * np.pi / (h * max(shape))) ** 2
    for precision, vtol, stol in (("fp64", 1e-12, 1e-10), ("mixed", 3e-6, 1e-6)):
        print("rows", shape, precision, flush=True)
        p = plan(shape, h, "periodic", precision)
        u, phi = empty(shape), empty(shape)
        assert p.solve_vacuum(dev(f), u) == gps.GPS_OK
        assert np.abs(host(u) - expect).max() <= vtol * np.abs(expect).max()
        assert p.solve_generalized(dev(f), dev(eps), phi, stol) == gps.GPS_OK
        err = np.linalg.norm(host(phi) - ref.phi)
        assert err <= 2.0 * stol * 4.0 * np.pi * np.linalg.norm(f) / lam
        p.close()
