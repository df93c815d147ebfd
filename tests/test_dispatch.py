"""Dispatch rules of the library's own entry points, asked of libgps.so on the CPU."""
import ctypes

import pytest

import test_index_bounds as ib
from paper_1509_00680_amd import gps
from test_fft_lengths import SPLITS, even_pairs


@pytest.mark.parametrize("L", sorted(SPLITS))
def test_row_pairs_depend_on_the_length_alone(L):
    """Row pairs per x-pass work-group: one count per length (a rule of its factors), at every
    number of rows and in both precisions."""
    a, b = SPLITS[L]
    P = ib.X_PAIRS(a) if L in ib.FAST else even_pairs(max(a, b))
    parts = gps.load()["_ZN3gps16fast_xpass_partsEii"]     # gps::fast_xpass_parts(int, int)
    parts.restype, parts.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.c_int]
    for rows in (4, 81, 900, 1024, 4095, 4096, 4097, 25600):
        assert parts(L, rows) == -(-((rows + 1) // 2) // P), rows
