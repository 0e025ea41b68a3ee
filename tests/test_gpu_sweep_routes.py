"""The sweep's launch forms against each other, bit for bit: several sweeps of a
single-workgroup lattice in one launch, eager neighbour reads for growth launches
of at most one workgroup per CU, and waves without cells in a small group.  The
512-thread mapping takes none of these routes (one launch per sweep, two cells per
thread) and is the reference; it is held to the oracle by the parity tests.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def states(sim, calls):
    out = []
    for n in calls:
        sim.sweep(n)
        out.append((sim.time(), sim.h0(), sim.width(), sim.get_lattice()))
    return out


# one workgroup: one block, 64 blocks of 32 x 32 (the most a group holds), 1024
# cells in two blocks, fewer cells than waves; 65 blocks and 1056 cells take two
@pytest.mark.parametrize("Lx,Ly", [(32, 32), (96, 96), (128, 128), (256, 256), (32, 2048), (32, 2080),
                                   (512, 128), (352, 192), (224, 224)])
@pytest.mark.parametrize("p,q,delayed", [(1.0, 0.0, 0), (0.7, 0.2, 0), (0.0, 1.0, 1), (0.9, 0.0, 1)])
def test_chained_sweeps_equal_single_launches(Lx, Ly, p, q, delayed):
    from paper_1110_6745_amd import okpz

    calls = [1, 2, 63, 65, 130]  # both copies current, one launch and several
    got = []
    for threads in (1024, 512):
        sim = okpz.okpz_init(Lx, Ly, p, q, 5 + Lx)
        sim.set_cell_borders(delayed)
        sim.set_threads(threads)
        got.append(states(sim, calls))
        sim.free()
    for a, b in zip(*got):
        assert a[:3] == b[:3] and np.array_equal(a[3], b[3]), f"t = {a[0]}"


# 255, 256 and 272 workgroups of 256 x 256 blocks, and small blocks
@pytest.mark.parametrize("Lx,Ly", [(4096, 4096), (4352, 4096), (3840, 4352), (1632, 1632), (2080, 1920)])
@pytest.mark.parametrize("copies", [1, 2])
def test_eager_reads_equal_gated_reads(Lx, Ly, copies):
    from paper_1110_6745_amd import okpz

    got = []
    for threads in (1024, 512):
        sim = (okpz.okpz_init if copies == 2 else okpz.okpz_init_in_place)(Lx, Ly, 1.0, 0.0, 3)
        sim.set_threads(threads)
        sim.sweep(7)
        got.append((sim.h0(), sim.width(), sim.get_lattice()))
        sim.free()
    assert got[0][:2] == got[1][:2] and np.array_equal(got[0][2], got[1][2])
