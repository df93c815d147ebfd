"""The plane pass (y forward, z and y inverse of the vacuum solver in one launch), restated on
the CPU: every step of k_plane with its index arithmetic, on the LDS tile, the half spectrum, the
reordered Green table and the partial sums, against numpy's transforms of the padded plane; every
index against its buffer; and the grids that take the pass."""
import numpy as np
import pytest

RADICES = (2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 15, 16)
LDS = 160 * 1024 - 512


def split(n, along_z, even):
    best, out = 17, None
    for x in range(2, 17):
        if n % x or x not in RADICES or (even and x % 2):
            continue
        y = n // x
        if (n > 5) if y == 1 else (y not in RADICES):
            continue
        m = max(x, y)
        if m < best or (m == best and along_z):
            best, out = m, (x, y)
    return out


def shape(ny, nz, pad_y, pad_z, elem=8):
    Ly, Lz = ny * (2 if pad_y else 1), nz * (2 if pad_z else 1)
    if Ly % 2:
        return None
    N = Ly // 2
    a, c = (split(N, False, False) if N >= 2 else None), split(Lz, True, pad_z)
    if a is None or c is None or c[1] == 1:
        return None
    PY = N | 1
    if (PY * Lz + Lz + 2 * N) * 2 * elem > LDS:
        return None
    return dict(N=N, nm=ny // N, Ly=Ly, Lz=Lz, A1=a[0], A2=a[1], C1=c[0], C2=c[1], PY=PY,
                ny=ny, nz=nz, pad_z=pad_z)


def root(n, e):
    return np.exp(-2j * np.pi * (np.asarray(e) % n) / n)


def dft(x, inverse):
    """Along axis 0, unnormalised."""
    return np.fft.ifft(x, axis=0) * len(x) if inverse else np.fft.fft(x, axis=0)


class Tile:
    """The LDS tile: reads and writes check their indices."""

    def __init__(self, s):
        self.a = np.full(s["PY"] * s["Lz"], np.nan + 0j)

    def read(self, i):
        assert i.min() >= 0 and i.max() < len(self.a)
        v = self.a[i]
        assert not np.isnan(v).any()               # written before it is read
        return v

    def write(self, i, v):
        i = np.broadcast_to(i, v.shape)
        assert i.min() >= 0 and i.max() < len(self.a)
        assert len(np.unique(i)) == i.size         # no two jobs write one element
        self.a[i] = v


def plane(s, half, table, r):
    """One work-group: half (nz, ny) of one kx, table[kz][position] of (kx, r)."""
    N, PY, A1, A2, C1, C2 = (s[k] for k in ("N", "PY", "A1", "A2", "C1", "C2"))
    nz, ny, Lz, Ly = s["nz"], s["ny"], s["Lz"], s["Ly"]
    t, src = Tile(s), half.reshape(-1)
    twz, twy, fold = root(Lz, np.arange(Lz)), root(N, np.arange(N)), root(Ly, np.arange(N))
    job = np.arange(nz * A2)
    z, n2 = job // A2, job % A2
    i = np.arange(A1)[:, None]
    x = src[z * ny + n2 + A2 * i]
    if s["nm"] == 2:
        v = src[z * ny + n2 + N + A2 * i]
        x = x - v if r else x + v
    if r:
        x = x * fold[A2 * i + n2]
    t.write(z * PY + n2 + A2 * i, dft(x, False) * twy[n2 * i])
    job = np.arange(nz * A1)
    k1, z = job // nz, job % nz
    i = np.arange(A2)[:, None]
    if A2 > 1:
        p = z * PY + A2 * k1 + i
        t.write(p, dft(t.read(p), False))
    job = np.arange(N * C2)
    q, y = job // N, job % N
    i = np.arange(C1)[:, None]
    p = (C2 * i + q) * PY + y
    rows = C1 // 2 if s["pad_z"] else C1
    x = np.zeros(p.shape, complex)
    x[:rows] = t.read(p[:rows])
    t.write(p, dft(x, False) * twz[q * i])
    job = np.arange(N * C1)
    k1, y = job // N, job % N
    i = np.arange(C2)[:, None]
    p = (C2 * k1 + i) * PY + y
    kz = k1 + C1 * i
    w = dft(t.read(p), False)
    x = w * table[np.minimum(kz, Lz - kz), y]
    delta = (x * w.conj()).real.sum()
    t.write(p, dft(x, True) * twz[i * k1].conj())
    job = np.arange(N * C2)
    q, y = job // N, job % N
    i = np.arange(C1)[:, None]
    p = (C2 * i + q) * PY + y
    x = dft(t.read(p), True)
    t.write(p[:rows], x[:rows])
    job = np.arange(nz * A1)
    k1, z = job // nz, job % nz
    i = np.arange(A2)[:, None]
    if A2 > 1:
        p = z * PY + A2 * k1 + i
        t.write(p, dft(t.read(p), True) * twy[i * k1].conj())
    job = np.arange(nz * A2)
    z, n2 = job // A2, job % A2
    i = np.arange(A1)[:, None]
    x = dft(t.read(z * PY + n2 + A2 * i), True)
    if r:
        x = x * fold[A2 * i + n2].conj()
    out = np.full(nz * N, np.nan + 0j)
    o = z * N + n2 + A2 * i
    assert len(np.unique(o)) == nz * N
    out[o] = x
    return out.reshape(nz, N), delta


GRIDS = [(3, 6), (2, 15), (5, 8), (24, 24), (45, 40), (32, 30), (63, 49), (81, 96), (96, 96),
         (27, 105), (64, 128), (100, 54)]


@pytest.mark.parametrize("ny,nz", GRIDS)
@pytest.mark.parametrize("pad_y", [True, False])
@pytest.mark.parametrize("pad_z", [True, False])
def test_steps_match_numpy(ny, nz, pad_y, pad_z):
    s = shape(ny, nz, pad_y, pad_z)
    if s is None:
        pytest.skip("no plane pass for this plane")
    rng = np.random.default_rng(ny * 1000 + nz)
    half = rng.normal(size=(nz, ny)) + 1j * rng.normal(size=(nz, ny))
    Ly, Lz, N = s["Ly"], s["Lz"], s["N"]
    green = rng.random((Lz // 2 + 1, Ly // 2 + 1))           # folded: [kz][ky]
    fz = np.minimum(np.arange(Lz), Lz - np.arange(Lz))
    fy = np.minimum(np.arange(Ly), Ly - np.arange(Ly))
    spec = np.fft.fft2(half, s=(Lz, Ly))
    full = green[np.ix_(fz, fy)]
    ref = (np.fft.ifft2(spec * full) * Lz * Ly)[:nz, :ny]
    pos = np.arange(N)
    kp = pos // s["A2"] + s["A1"] * (pos % s["A2"])
    assert sorted(kp) == list(range(N))
    parts, delta = [], 0.0
    for r in (0, 1):
        ky = r + 2 * kp
        y, d = plane(s, half, green[:, np.minimum(ky, Ly - ky)], r)
        parts.append(y)
        delta += d
    y = np.arange(ny)
    got = np.where(y >= N, parts[0][:, y % N] - parts[1][:, y % N],
                   parts[0][:, y % N] + parts[1][:, y % N])
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
    assert abs(delta / (full * np.abs(spec) ** 2).sum() - 1.0) <= 1e-12


def test_partial_sums_cover_every_row_once():
    """The x inverse reads row (z, y) at z N + y - m N of both partial sums, m = y >= N, and the
    partial arrays hold nz N values per plane and parity: Ly nz Kx in all, the work buffer."""
    for ny, nz in GRIDS:
        for pad_y in (True, False):
            s = shape(ny, nz, pad_y, True)
            if s is None:
                continue
            assert s["nm"] == (1 if pad_y else 2) and s["nm"] * s["N"] == ny
            assert 2 * s["N"] * nz == s["Ly"] * nz
            row = np.arange(ny * nz)
            z, y = row // ny, row % ny
            off = z * s["N"] + np.where(y >= s["N"], y - s["N"], y)
            assert off.min() >= 0 and off.max() < nz * s["N"]
            assert (np.bincount(off) == s["nm"]).all()
