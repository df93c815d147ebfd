"""The rule by which a grid takes the plane pass (plane_shape in gps_fft.hip), restated in full:
the route of vacuum solves, SC/PSD steps and PCG solves on a grid, and what it takes of a plan's
memory."""
import test_index_bounds as ib
from test_fft_lengths import SPLITS, even_pairs
from test_plane_pass import LDS, split

MAX_LX, MAX_GROUP = 200, 1100
VACUUM_POINTS, SOLVE_POINTS, FEW_POINTS, SOLVE_VALUES = 5000000, 3500000, 1500000, 209


def lengths(shape, bc):
    nz, ny, nx = shape
    pxy, pz = bc in ("surface", "periodic"), bc in ("periodic", "wire")
    return (nx if pxy else 2 * nx), (ny if pxy else 2 * ny), (nz if pz else 2 * nz)


def row_pairs(L, rows=None, elem=8):
    """Row pairs of an x-pass work-group; rows None: a grid of many rows."""
    a, b = SPLITS[L]
    if elem == 4 and L <= 64 and rows is not None and rows <= 4096:
        return 4
    return ib.X_PAIRS(a) if L in ib.FAST else even_pairs(max(a, b))


def xinv_values(L, lout, periodic):
    """Values that a thread of the solve's x inverse holds (its operands, row loads, twiddles and
    shares of the partial sums)."""
    P = row_pairs(L)
    nt = ib.round64(P * max(SPLITS[L]))
    kp = -(-(L // 2 + 1) // (nt // P))
    out = -(-2 * P * lout // nt)
    shares = (16 if nt == 64 else 8) * (2 if periodic else 1)
    return 8 * kp + (6 if periodic else 5) * out + 2 * -(-L // nt) + 2 * shares


def two_level_solve(L, lout, elem, six):
    """Whether PCG solves on rows of lout points (FFT length L) run the two-level x passes; six: the
    x inverse reads six fields (refinement, the periodic mean term), not five."""
    if L not in SPLITS:
        return False
    if elem == 4 or not six or lout != L:
        return True
    P = row_pairs(L)
    nt = ib.round64(P * max(SPLITS[L]))
    rows, points = P * -(-(L // 2 + 1) // nt), -(-2 * P * lout // nt)
    return 2 * (4 * rows + 6 * points) < 528


def plane(shape, bc, elem):
    """(vacuum solves and SC/PSD steps, PCG solves) take the plane pass; elem: 4 FP32, 8 FP64."""
    nz, ny, nx = shape
    Lx, Ly, Lz = lengths(shape, bc)
    n = nx * ny * nz
    if Lx not in SPLITS or Lx > MAX_LX or Ly % 2 or Ly < 4 or n > VACUUM_POINTS:
        return False, False
    N = Ly // 2
    z = split(Lz, True, bc in ("free", "surface"))
    if split(N, False, False) is None or z is None or z[1] == 1:
        return False, False
    lds = ((N | 1) * Lz + Lz + 2 * N) * 2 * elem
    if lds > LDS or lds > MAX_GROUP * 2 * (Lx // 2 + 1):
        return False, False
    values = xinv_values(Lx, nx, bc == "periodic")
    return True, elem == 4 and n <= SOLVE_POINTS and (n <= FEW_POINTS or values <= SOLVE_VALUES)
