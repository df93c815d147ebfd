"""Dispatch rules of the library's own entry points, asked of libgps.so on the CPU."""
import ctypes

import numpy as np
import pytest

import plane_rule
from test_plane_memory import needs_host, run_host
from paper_1509_00680_amd import gps
from test_fft_lengths import SPLITS


@pytest.mark.parametrize("L", sorted(SPLITS))
@pytest.mark.parametrize("elem", [4, 8])
def test_row_pairs(L, elem):
    """Row pairs per x-pass work-group: by the length's factors, but four in FP32 at every length
    up to 64 on grids of up to 4096 rows."""
    # gps::fast_xpass_parts<T>(int, int)
    parts = gps.load()["_ZN3gps16fast_xpass_partsI%sEEiii" % {4: "f", 8: "d"}[elem]]
    parts.restype, parts.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int]
    for rows in (4, 81, 900, 1024, 4095, 4096, 4097, 25600):
        P = plane_rule.row_pairs(L, rows, elem)
        assert parts(L, rows) == -(-((rows + 1) // 2) // P), rows


def _footprint(shape, bc, precision, compact=False):
    """(tables, buffers) of one PCG solve, of a plan with or without the plane pass."""
    lib = gps.load()
    f = lib["_ZN3gps22compact_plan_footprintEiiiiiiiiPmS0_S0_"] if compact else \
        lib.gps_plan_footprint
    t, b = ctypes.c_size_t(), ctypes.c_size_t()
    nz, ny, nx = shape
    assert f(ctypes.c_int(nx), ctypes.c_int(ny), ctypes.c_int(nz),
             ctypes.c_int(gps.BC_CODES[bc]), ctypes.c_int(gps.PRECISIONS[precision]),
             ctypes.c_int(100), ctypes.c_int(0), ctypes.c_int(0), ctypes.byref(t),
             ctypes.byref(b), None) == gps.GPS_OK
    return t.value, b.value


def _smooth(n):
    for f in (2, 3, 5, 7):
        while n % f == 0:
            n //= f
    return n == 1


EXTENTS = [n for n in range(2, 321) if _smooth(n)]


@pytest.mark.parametrize("bc", ["free", "surface", "periodic", "wire"])
def test_plane_pass_rule(bc):
    """The footprint shows which grids have the pass (its tables) and which PCG solves take it
    (their half spectrum): the rule restated in plane_rule, over grids of every size."""
    rng = np.random.default_rng(17)
    grids = [tuple(int(v) for v in rng.choice(EXTENTS, 3)) for _ in range(3000)]
    grids += [(n, n, n) for n in EXTENTS]
    took = {4: 0, 8: 0, "solve": 0}
    for shape in grids:
        Lx, Ly, Lz = plane_rule.lengths(shape, bc)
        entries = (Lx // 2 + 1) * Ly * (Lz // 2 + 1)
        half = shape[0] * shape[1] * (Lx // 2 + 1) * 8
        vac32, pcg32 = plane_rule.plane(shape, bc, 4)
        vac64, pcg64 = plane_rule.plane(shape, bc, 8)
        assert not pcg64
        for precision, solve in (("mixed", pcg32), ("fp64", False)):
            t, b = _footprint(shape, bc, precision)
            t0, b0 = _footprint(shape, bc, precision, compact=True)
            assert t - t0 == entries * (4 * vac32 + 8 * vac64), (shape, precision)
            assert b - b0 == solve * half, (shape, precision)
        took[4] += vac32
        took[8] += vac64
        took["solve"] += pcg32
    assert min(took.values()) > 20


@pytest.mark.parametrize("shape,bc", [((192, 192, 192), "periodic"), ((120, 120, 120), "periodic"),
                                      ((180, 180, 180), "periodic"), ((64, 300, 200), "surface")])
def test_solves_that_the_pass_slows_down_keep_the_three_passes(shape, bc):
    """Measured 2 to 15 % slower with the plane pass than with the y, z and y passes."""
    assert _footprint(shape, bc, "mixed")[1] == _footprint(shape, bc, "mixed", compact=True)[1]


@needs_host
def test_x_passes_of_solves_on_full_rows():
    """Which x passes PCG solves launch, at every length, counted on the host."""
    r = run_host("x_routes.cpp")
    assert r.returncode == 0, r.stderr[-2000:]
    generic = set()
    for line in r.stdout.splitlines():
        L, bc, precision, refine, route = line.split()
        L, six = int(L), bc == "periodic" or refine != "0"
        fast = plane_rule.two_level_solve(L, L, {"fp64": 8, "mixed": 4}[precision], six)
        assert route == ("two-level" if fast else "generic"), line
        if L in SPLITS and not fast:
            generic.add((L, precision))
    assert generic == {(L, "fp64") for L in (324, 378, 400, 420, 432)}
