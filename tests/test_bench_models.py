"""bench.py's byte models against the arrays that the kernels read and write, counted one by one."""
import os
import sys
from types import SimpleNamespace

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
bench = pytest.importorskip("bench")

W = SimpleNamespace(n_vox=30, M=32, K=28, n_views=7, ewald=1, geometry="axis")


def test_slice_path_bytes():
    columns = 17                                           # kx = 0 .. M / 2 of every row frequency
    images, filt, q = 4 * 32 * 32, 16 * 32 * columns, 16 * 32 * columns
    partial = 4 * 32 * 30 * 30                             # M real slices of N x N
    assert bench.slice_bytes("spectra", W) == 7 * (images + filt + q)
    assert bench.slice_bytes("planes", W) == 7 * q + partial
    assert bench.slice_bytes("grid", W) == partial + 4 * 30 ** 3


@pytest.mark.parametrize("mode", [1, 2])
def test_fourier_form_bytes(mode):
    images, filt, q = 4 * 32 * 32, 8 * 32 * 32, 8 * 32 * 32     # complex filter and spectra
    assert bench.algorithmic_bytes("spectra", W, 7, True, fourier_mode=mode) == 7 * (images + filt + q)
    vertices, cells = 31 ** 3, 30 ** 3
    got = bench.algorithmic_bytes("fgrid", W, 7, True, fourier_mode=mode, entries=1000)
    if mode == 1:       # entries, row offsets, spectra and sampling matrix read, complex grid written
        assert got == 8 * 1000 + 4 * vertices + 7 * q + 8 * cells + 8 * cells
    else:               # spectra read, accumulator (two 64-bit integers) cleared and updated
        assert got == 7 * q + 2 * 16 * vertices


def test_stack_path_bytes():
    images, filt, q = 4 * 32 * 32, 16 * 32 * 32, 16 * 32 * 32
    assert bench.algorithmic_bytes("spectra", W, 7, True) == 7 * (images + filt + q)
