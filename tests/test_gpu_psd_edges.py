"""Spectrum where its kernels' tilings end, with the tolerance of the spectrum
parity tests: strips of 8192 columns with one word more or less, rows that are no
multiple of a lane's four words, runs shorter than a carry-save group and a last
workgroup with few rows, transforms of one tile, of one to five wide stages, and one
axis of each kind.
"""
import numpy as np
import pytest

import oracle
from tests import inputs
from tests.test_gpu_psd import check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def okpz():
    from paper_1110_6745_amd import okpz as m

    return m


@pytest.mark.parametrize("Lx,Ly", [(8192, 64), (8224, 32), (8160, 96), (16384, 32), (24640, 32), (160, 2080),
                                   (4096, 1024), (4128, 64), (64, 4064), (2016, 2080), (32768, 96), (65536, 32),
                                   (33 * 32, 16384), (128, 32800)])
@pytest.mark.parametrize("copies", [1, 2])
def test_spectrum_at_tile_edges(okpz, Lx, Ly, copies):
    lat, H0 = inputs.rough_state(Lx, Ly, seed=Lx + Ly, mcs=1)
    sim = (okpz.okpz_init if copies == 2 else okpz.okpz_init_in_place)(Lx, Ly, 0.9, 0.2, 3)
    sim.set_lattice(lat, H0, 7)
    check(sim.psd(), lat, H0, f"{Lx}x{Ly} as loaded")
    sim.sweep(2)  # two copies: rotated columns, column 0 inside a strip
    H = oracle.run(lat, 0.9, 0.2, 3, 7, 2, H0)
    check(sim.psd(), lat, H, f"{Lx}x{Ly} after 2 sweeps")
    a, b = sim.psd(), sim.psd_noalloc()
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    sim.free()


def test_steep_rows_fill_the_row_sums(okpz):
    # one hill over the whole row: the largest row sums and differences of a strip
    Lx, Ly = 65536, 64
    a = np.zeros(Lx, dtype=np.uint8)
    a[Lx // 4:3 * Lx // 4] = 1
    lat = inputs.separable_rows(a, inputs.balanced_bits(Ly, 4), 0, Ly)
    sim = okpz.okpz_init(Lx, Ly, 1.0, 0.0, 1)
    sim.set_lattice(lat, 0, 0)
    check(sim.psd(), lat, 0, "hill")
    sim.free()
