"""The two-level FFT lengths: which lengths have them, their splits, and the
bounds of their strided passes, replayed on the CPU from the splits in the
sources."""
import os
import re

import numpy as np
import pytest

import test_index_bounds as ib

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1509_00680_amd", "csrc")


def splits():
    out = {}
    for name, macro in (("gps_fft_fast.hip", "GPS_TUNED_LENGTH"),
                        ("gps_fft_lengths.hip", "GPS_LENGTH")):
        text = open(os.path.join(CSRC, name)).read()
        for a, b in re.findall(r"^%s\((\d+), (\d+)\)" % macro, text, re.M):
            L = int(a) * int(b)
            assert L not in out, L
            out[L] = (int(a), int(b))
    return out


SPLITS = splits()


def smooth(n):
    for f in (2, 3, 5, 7):
        while n % f == 0:
            n //= f
    return n == 1


def even_pairs(m):
    best = 6
    for P in range(5, 11):
        if P * m * ib.round64(best * m) > best * m * ib.round64(P * m):
            best = P
    return best


def test_lengths_and_splits():
    assert SPLITS == {L: SPLITS[L] for L in range(2, 449) if smooth(L) and
                      ((L % 2 == 0 and L >= 16) or (L % 2 and 15 <= L <= 225))}
    for L, (a, b) in SPLITS.items():
        assert L % 2 or a % 2 == 0, L          # the padded half is a half of L1
    text = open(os.path.join(CSRC, "gps_fft_reg.h")).read()
    codelets = {int(n) for n in re.findall(r"^GPS_(?:PFA_)?CODELET\((\d+),", text, re.M)}
    assert {f for s in SPLITS.values() for f in s} <= codelets


def violations(T, mode, L, Lin, Lout, npen, per_group, group_stride, elem_stride, wsize, Kx=None,
               Ly=None, tabsize=None, decide=False):
    L1, L2 = SPLITS[L]
    B = 8 if T == "d" or L >= 320 else 16
    pad = L1 % 2 == 0 and (
        (mode == ib.ST_FWD and 2 * Lin == L) or
        (mode == ib.ST_CONV and 2 * Lin == L and Lout == Lin) or
        (mode == ib.ST_INV and 2 * Lout == L and Lin == L))
    NT = ib.round64(B * max(L1, L2))
    groups = (npen + B - 1) // B
    # partial sums of the z pass: one per wavefront
    if mode == ib.ST_CONV and groups * (NT // 64) > npen + 64:
        return ["partials"]
    dec = 1 if decide else 0
    bid = np.arange(dec, groups + dec)[:, None]
    tid = np.arange(NT)[None, :]
    b, q = tid & (B - 1), tid // B
    tile = ib.xcd_tile(bid, groups + dec) - dec
    return ib._tile(T, mode, L, Lin, Lout, npen, per_group, group_stride, elem_stride, wsize,
                    Kx, Ly, tabsize, True, tile * B + b, q, L1, L2, pad)


@pytest.mark.parametrize("L", sorted(SPLITS))
def test_strided_passes_in_bounds(L):
    """The length on the y and on the z axis, padded and full, beside short axes."""
    n = 0
    for pad in ((True, False) if L % 2 == 0 else (False,)):
        box = L // 2 if pad else L
        for shape in ((5, box, 9), (box, 3, 9)):
            for tag, T, args, kw in ib.launches(shape, "free" if pad else "periodic"):
                if args[1] != L:
                    continue
                for decide in ((False, True) if tag == "y inverse" else (False,)):
                    assert not violations(T, *args, decide=decide, **kw), (shape, tag, T)
                n += 1
    assert n > 0


@pytest.mark.parametrize("L,few", [(L, False) for L in sorted(SPLITS)] +
                         [(L, True) for L in (32, 48, 64)])
def test_x_pass_tiles_cover_the_rows(L, few):
    """Every element of a tile is loaded by exactly one (thread, step), and the
    row and column the kernel advances by addition are those of the division."""
    L1, L2 = SPLITS[L]
    tuned = L in ib.FAST
    P = 4 if few else ib.X_PAIRS(L1) if tuned else even_pairs(max(L1, L2))
    NT = ib.round64(P * max(L1, L2))
    assert NT <= 512
    for width in ((L // 2, L) if L % 2 == 0 else (L,)):
        steps = (2 * P * width + NT - 1) // NT
        tid = np.arange(NT)
        row, col = tid // width, tid % width
        for i in range(steps):
            e = tid + i * NT
            np.testing.assert_array_equal(row * width + col, e)
            assert (col < width).all()
            col = col + NT % width
            row = row + NT // width
            wrap = col >= width
            col, row = np.where(wrap, col - width, col), np.where(wrap, row + 1, row)
        assert steps * NT >= 2 * P * width
    # the transform's threads: q < L2 in one step and q < L1 in the other
    assert P * max(L1, L2) <= NT
