"""GPU parity of the solver on grids around the plane pass's limits, against the FP64 oracle:
odd, even, smallest and largest planes, each boundary condition, both precisions; the same x
lengths without the pass (nz = 2 has none); and a served request whose budget leaves no room for
it.  Tolerances of the parity tests: vacuum 1e-12 (FP64) and 3e-6 (mixed) of max|u|, solves 1e-8
max|phi| (FP64) and 1e-5 (mixed)."""
import numpy as np
import pytest

from oracle import green, pb, pcg
from paper_1509_00680_amd import gps
from paper_1509_00680_amd import workloads as W
from gpu_util import dev, host, empty, oracle_ions, plan, require_gpu

pytestmark = pytest.mark.gpu

# (nz, ny, nx): the last four are the largest FP32 and FP64 tiles, free and periodic in plane
SHAPES = [(3, 3, 8), (8, 9, 15), (15, 2, 16), (21, 16, 25), (96, 96, 50), (64, 64, 32),
          (128, 128, 64), (64, 128, 63), (2, 5, 30)]


@pytest.mark.parametrize("bc", ["free", "surface", "periodic", "wire"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_vacuum(shape, bc, precision):
    require_gpu()
    rng = np.random.default_rng(5)
    f = rng.normal(size=shape)
    if bc == "periodic":
        f -= f.mean()
    expect = green.VacuumSolver(shape, 0.45, bc).apply(f)
    p = plan(shape, 0.45, bc, precision)
    u = empty(shape)
    print("plane vacuum", shape, bc, precision, flush=True)
    for _ in range(2):
        assert p.solve_vacuum(dev(f), u) == gps.GPS_OK
        tol = 1e-12 if precision == "fp64" else 3e-6
        assert np.abs(host(u) - expect).max() <= tol * np.abs(expect).max()


def _problem(shape, bc, seed):
    rng = np.random.default_rng(seed)
    z, y, x = np.meshgrid(*[2.0 * np.pi * np.arange(m) / m for m in shape], indexing="ij")
    eps = 6.0 + 2.0 * np.cos(x) * np.cos(y) + np.sin(z)
    rho = rng.normal(size=shape)
    if bc == "periodic":
        rho -= rho.mean()
    return rho, eps


@pytest.mark.parametrize("bc", ["free", "surface", "periodic", "wire"])
@pytest.mark.parametrize("shape", [(3, 3, 8), (8, 9, 15), (21, 16, 25), (20, 27, 24), (2, 5, 30)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves(shape, bc, precision):
    """Generalized Poisson and, with the periodic k = 0 multiplier, linear Poisson-Boltzmann."""
    require_gpu()
    rho, eps = _problem(shape, bc, 7)
    p = plan(shape, 0.5, bc, precision)
    phi = empty(shape)
    tol = 1e-11 if precision == "fp64" else 1e-6
    bound = 1e-8 if precision == "fp64" else 1e-5
    print("plane solve", shape, bc, precision, flush=True)
    ref = pcg.pcg_solve(rho, eps, 0.5, bc, tol=1e-11)
    assert p.solve_generalized(dev(rho), dev(eps), phi, tol) == gps.GPS_OK
    assert np.abs(host(phi) - ref.phi).max() <= bound * np.abs(ref.phi).max()
    ions = W.electrolyte_1to1(W.debye_concentration(3.0), linear=True)
    ref = pb.solve_linear_pb(rho, eps, 0.5, bc, oracle_ions(ions), 1e-11)
    for _ in range(2):                            # the second solve starts from used buffers
        assert p.solve_pb(dev(rho), dev(eps), ions, phi, tol) == gps.GPS_OK
        assert np.abs(host(phi) - ref.phi).max() <= bound * np.abs(ref.phi).max()


@pytest.mark.parametrize("slots", [1, 2])
def test_budget_without_room_for_the_plane_pass(slots):
    require_gpu()
    n, h = 24, 0.5
    prob = W.molecule(n, h, seed=3, n_atoms=6, ball=2.0)
    tables, buffers, transient = gps.plan_footprint(prob.shape, "free", "mixed")
    table = (n + 1) * 2 * n * (n + 1)             # reordered spectrum, FP32 and FP64 copies
    half = n * n * (n + 1) * 8                    # half spectrum along x, FP32 complex
    budget = tables - 12 * table + slots * (buffers - half) + transient
    srv = gps.Server(budget_bytes=budget, max_active=1, precision="mixed", batch_slots=slots)
    phi = empty(prob.shape)
    rho, eps = dev(prob.rho), dev(prob.eps)
    print("plane budget", slots, flush=True)
    st, t = srv.submit(rho, eps, phi, h, "free", 1e-6)
    assert st == gps.GPS_OK, gps.STATUS[st]
    assert srv.wait(t)["status"] == gps.GPS_OK
    assert srv.stats()["bytes_peak"] <= budget
    srv.close()
    small = gps.Server(budget_bytes=budget - 1, max_active=1, precision="mixed",
                       batch_slots=slots)
    st, _ = small.submit(rho, eps, phi, h, "free", 1e-6)
    assert st == gps.GPS_E_NOMEM                  # as it was: nothing smaller would do
    small.close()
    ref = pcg.pcg_solve(prob.rho, prob.eps, h, "free", tol=1e-10)
    assert np.abs(host(phi) - ref.phi).max() <= 1e-5
