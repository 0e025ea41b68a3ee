"""Exact width sums where the width kernels' tilings end: rows of less than a lane's
four words, of one pass (256 words) and one word more, unaligned rows, a rotation
inside each word of a lane, runs of one row and of several per wavefront, and steep
surfaces that fill the chunk table's fields.
"""
import numpy as np
import pytest

import oracle
from tests import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def okpz():
    from paper_1110_6745_amd import okpz as m

    return m


def hill(L):
    """Up for half the lattice, then down: the steepest closed walk."""
    a = np.zeros(L, dtype=np.uint8)
    a[:L // 2] = 1
    return a


@pytest.mark.parametrize("Lx,Ly", [(32, 32), (64, 32), (96, 64), (128, 32), (160, 96), (8160, 64),
                                   (8192, 32), (8224, 32), (16384, 96), (24608, 32)])
@pytest.mark.parametrize("shape", ["hill", "random"])
def test_width_of_closed_walks(okpz, Lx, Ly, shape):
    if shape == "hill":
        a, b = hill(Lx), hill(Ly)
    else:
        a, b = inputs.balanced_bits(Lx, 5), inputs.balanced_bits(Ly, 6)
    lat = inputs.separable_rows(a, b, 0, Ly)
    sim = okpz.okpz_init(Lx, Ly, 1.0, 0.0, 1)
    for H0 in (0, -4):
        sim.set_lattice(lat, H0, 0)
        assert sim.width() == oracle.width_sums(lat, H0)
    sim.free()


@pytest.mark.parametrize("Lx,Ly", [(256, 256), (1056, 96), (8448, 64)])
def test_width_under_rotation(okpz, Lx, Ly):
    sim = okpz.okpz_init(Lx, Ly, 0.8, 0.1, 9)
    for _ in range(12):  # each sweep stores the columns at another rotation
        sim.sweep(1)
        assert sim.width() == oracle.width_sums(sim.get_lattice(), sim.h0())
    sim.free()


# more rows than one run per wavefront (8192 rows), not a multiple of a run
@pytest.mark.parametrize("Ly", [8192, 8224, 32768, 50016])
def test_width_of_many_rows(okpz, Ly):
    a, b = inputs.balanced_bits(64, 2), inputs.balanced_bits(Ly, 3)
    lat = inputs.separable_rows(a, b, 0, Ly)
    sim = okpz.okpz_init(64, Ly, 1.0, 0.0, 1)
    sim.set_lattice(lat, 2, 0)
    assert sim.width() == oracle.width_sums(lat, 2)
    sim.free()
