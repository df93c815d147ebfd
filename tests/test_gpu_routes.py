"""GPU parity on grids chosen by their route, each asserted from the restated rule: SC and PSD
steps whose stop decisions run in the two-level y inverse, in the generic one and in the plane
pass; the x passes of every full row length beside the plane pass and without it; and the
largest tiles of the plane pass.

Solves are compared after three PCG iterations with the oracle's third iterate: on these cells,
many times longer than wide, a converged FP32 solution is as far from the true one as the cell is
ill-conditioned, while the iterates depend on every pass and epilogue and stay within the 1e-5 of
max|phi| that mixed solves are held to.  Vacuum solves: 1e-12 (FP64) and 3e-6 (mixed) of
max|u|; SC and PSD iterates: 1e-10 and 1e-5 of max|phi|."""
import numpy as np
import pytest

import plane_rule
from oracle import green, pcg, sc
from paper_1509_00680_amd import gps
from gpu_util import dev, host, empty, plan, require_gpu
from test_fft_lengths import SPLITS

pytestmark = pytest.mark.gpu

VACUUM_TOL = {"fp64": 1e-12, "mixed": 3e-6}
ELEM = {"fp64": 8, "mixed": 4}


def _fields(shape, bc, seed):
    rng = np.random.default_rng(seed)
    z, y, x = np.meshgrid(*[2.0 * np.pi * np.arange(m) / m for m in shape], indexing="ij")
    eps = 6.0 + 2.0 * np.cos(x) * np.cos(y) + np.sin(z)
    rho = rng.normal(size=shape)
    if bc == "periodic":
        rho -= rho.mean()
    return rho, eps


def _vacuum(shape, bc, precision, f, expect):
    p = plan(shape, 0.45, bc, precision)
    u = empty(shape)
    assert p.solve_vacuum(dev(f), u) == gps.GPS_OK
    assert np.abs(host(u) - expect).max() <= VACUUM_TOL[precision] * np.abs(expect).max()
    p.close()


def _three_iterations(shape, bc, precision, rho, eps, **kw):
    ref = pcg.pcg_solve(rho, eps, 0.45, bc, tol=1e-30, maxit=3)
    p = plan(shape, 0.45, bc, precision, maxit=3, **kw)
    phi = empty(shape)
    assert p.solve_generalized(dev(rho), dev(eps), phi, 1e-30) == gps.GPS_E_NOT_CONVERGED
    assert p.info()["iterations"] == 3
    bound = 1e-8 if precision == "fp64" else 1e-5
    assert np.abs(host(phi) - ref.phi).max() <= bound * np.abs(ref.phi).max()
    p.close()


# shape, boundary condition, the y pass (None: the plane pass)
SC_GRIDS = [((18, 6, 7), "free", "generic"), ((6, 6, 105), "free", "generic"),
            ((9, 15, 105), "free", "two-level"), ((48, 64, 20), "free", "two-level"),
            ((10, 15, 16), "surface", "two-level"), ((5, 7, 16), "surface", "generic"),
            ((18, 6, 10), "free", None), ((9, 15, 16), "wire", None)]


@pytest.mark.parametrize("shape,bc,route", SC_GRIDS)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_sc_and_psd_steps_by_route(shape, bc, route, precision):
    require_gpu()
    Ly = plane_rule.lengths(shape, bc)[1]
    taken = plane_rule.plane(shape, bc, ELEM[precision])[0]
    assert taken == (route is None)
    assert route is None or (Ly in SPLITS) == (route == "two-level")
    rng = np.random.default_rng(41)
    z, y, x = np.meshgrid(*[np.linspace(-1.0, 1.0, n) for n in shape], indexing="ij")
    rho = rng.normal(size=shape)
    eps = 1.0 + 30.0 / (1.0 + np.exp(-6.0 * (z * z + y * y + x * x - 0.6)))
    for steps in (1, 2, 7):
        pl = plan(shape, 0.5, bc, precision, maxit=steps)
        phi = empty(shape)
        for method in ("sc", "psd", "psd_weighted", "sc"):
            if method == "sc":
                ref, _, _ = sc.sc_solve(rho, eps, 0.5, bc, 0.6, tol=0.0, maxit=steps)
            else:
                ref, _, _ = sc.psd_solve(rho, eps, 0.5, bc, tol=0.0, maxit=steps,
                                         step="paper" if method == "psd" else "weighted")
            print("sc route", shape, bc, route, precision, steps, method, flush=True)
            st = pl.solve_sc(dev(rho), dev(eps), phi, 1e-30, method=method, eta=0.6)
            assert st == gps.GPS_E_NOT_CONVERGED, gps.STATUS[st]
            assert pl.info()["iterations"] == steps
            bound = 1e-10 if precision == "fp64" else 1e-5
            assert np.abs(host(phi) - ref).max() <= bound * np.abs(ref).max()
        pl.close()


@pytest.mark.parametrize("L", sorted(SPLITS))
def test_full_rows_beside_both_routes(L):
    """Rows of L points along x (periodic, with the mean term): beside the plane pass up to its
    longest x length, and beside the y, z and y passes."""
    require_gpu()
    for nz, with_plane in ((6, L <= plane_rule.MAX_LX), (2, False)):
        shape = (nz, 4, L)
        assert plane_rule.plane(shape, "periodic", 4) == (with_plane, with_plane)
        assert plane_rule.plane(shape, "periodic", 8)[0] == with_plane
        rho, eps = _fields(shape, "periodic", L)
        expect = green.VacuumSolver(shape, 0.45, "periodic").apply(rho)
        for precision in ("fp64", "mixed"):
            print("full rows", shape, precision, flush=True)
            _vacuum(shape, "periodic", precision, rho, expect)
            _three_iterations(shape, "periodic", precision, rho, eps)


@pytest.mark.parametrize("L", [L for L in sorted(SPLITS) if L <= 64])
def test_short_rows_on_both_sides_of_the_row_count(L):
    """Up to 64 points a row the FP32 x passes take four row pairs per work-group on few rows and
    the length's own count on many; full and padded rows."""
    require_gpu()
    for bc, n in (("periodic", L),) + ((("free", L // 2),) if L % 2 == 0 else ()):
        for shape, few in (((63, 64, n), True), ((70, 60, n), False)):
            rows = shape[0] * shape[1]
            assert (plane_rule.row_pairs(L, rows, 4) == 4) == few
            rho, eps = _fields(shape, bc, L)
            expect = green.VacuumSolver(shape, 0.45, bc).apply(rho)
            print("rows", shape, bc, flush=True)
            _vacuum(shape, bc, "mixed", rho, expect)
            _three_iterations(shape, bc, "mixed", rho, eps)


@pytest.mark.parametrize("L", [32, 63, 200, 225, 320, 324, 360, 378, 400, 420, 432, 448])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_tracked_solves_on_full_rows(L, precision):
    """Three iterations that carry the FP64 source of the iterate (refinement on, its first
    recomputation past the end), on full rows whose x passes are the two-level ones and (FP64,
    five long lengths) the generic ones."""
    require_gpu()
    shape, bc = (6, 4, L), "surface"
    fast = plane_rule.two_level_solve(L, L, ELEM[precision], True)
    assert fast == (precision == "mixed" or L not in (324, 378, 400, 420, 432))
    rho, eps = _fields(shape, bc, L)
    print("tracked rows", shape, precision, flush=True)
    _three_iterations(shape, bc, precision, rho, eps, refine_every=100)


# shape, boundary condition, element, PCG solves take it
TILES = [((96, 96, 80), "free", 4, True), ((98, 98, 98), "free", 4, True),
         ((64, 64, 64), "free", 8, False), ((63, 63, 63), "free", 8, False),
         ((98, 98, 90), "wire", 8, False), ((98, 200, 160), "surface", 4, True),
         ((128, 128, 128), "periodic", 8, False), ((112, 112, 112), "periodic", 4, True),
         ((196, 180, 140), "periodic", 4, False)]


@pytest.mark.parametrize("shape,bc,elem,solve", TILES)
def test_largest_tiles(shape, bc, elem, solve):
    require_gpu()
    assert plane_rule.plane(shape, bc, elem) == (True, solve)
    rho, eps = _fields(shape, bc, 3)
    precision = "mixed" if elem == 4 else "fp64"
    print("tile", shape, bc, precision, flush=True)
    expect = green.VacuumSolver(shape, 0.45, bc).apply(rho)
    _vacuum(shape, bc, precision, rho, expect)
    if solve:
        _three_iterations(shape, bc, precision, rho, eps)
