"""H0 = h(0,0) through many sweeps, whose random shifts put site (0,0) into every
32-site piece of its block row: the kernels count the bonds of the row's prefix
piece by piece.  Exact against the oracle, for block sides 32 to 256, one block
and several, both thread-cell borders and one lattice copy or two.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Lx,Ly", [(32, 32), (256, 64), (256, 256), (96, 160), (512, 128)])
@pytest.mark.parametrize("p,q", [(1.0, 0.0), (0.6, 0.4), (0.7, 0.0), (0.0, 1.0)])
@pytest.mark.parametrize("delayed,copies", [(0, 2), (1, 1)])
def test_h0_over_many_shifts(Lx, Ly, p, q, delayed, copies):
    from paper_1110_6745_amd import okpz

    seed, sweeps = 11 + Lx + Ly, 40
    sim = (okpz.okpz_init if copies == 2 else okpz.okpz_init_in_place)(Lx, Ly, p, q, seed)
    sim.set_cell_borders(delayed)
    lat, H0 = oracle.flat(Lx, Ly), 0
    for s in range(sweeps):
        sim.sweep(1)
        H0 = oracle.sweep(lat, p, q, seed, s, H0, delayed=bool(delayed))
        assert sim.h0() == H0, f"after sweep {s}"
    assert np.array_equal(sim.get_lattice(), lat)
    sim.free()
