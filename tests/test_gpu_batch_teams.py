"""Jobs whose workgroups stay with them from sweep to sweep, against the same jobs run
alone: two to sixteen items per sweep (not all of one size), claims of one and of two
items, more and fewer workgroups than items (teams of all jobs, of some, of none),
samples measured by the team's members, slices that end a team between two sweeps, the
last sweep with and without a sample, both thread-cell borders.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# sides, sweeps: 16, 16, 9, 13, 2, 4, 1 and 2 items per sweep, 63 in all
SIZES = [(1024, 1024, 45), (256, 4096, 33), (768, 768, 61), (896, 896, 40), (512, 256, 101), (448, 448, 70),
         (128, 96, 90), (8192, 32, 37)]


def alone(okpz, job, borders, m):
    Lx, Ly, p, q, seed, t_max = job
    sim = okpz.okpz_init(Lx, Ly, p, q, seed)
    sim.set_cell_borders(borders)
    out = [(t, *sim.width(t)) for t in okpz.sampling_times(t_max, m)]
    sim.sweep(t_max - sim.time())
    res = out, sim.h0(), sim.get_lattice()
    sim.free()
    return res


@pytest.mark.parametrize("p,q,borders", [(1.0, 0.0, 0), (0.8, 0.1, 0), (1.0, 0.0, 1)])
def test_teams(p, q, borders):
    from paper_1110_6745_amd import okpz

    m = 0.03
    jobs = [(Lx, Ly, p, q, 11 * i + 3, t) for i, (Lx, Ly, t) in enumerate(SIZES)]
    refs = [alone(okpz, j, borders, m) for j in jobs]
    b = okpz.Batch(jobs, m)
    b.set_cell_borders(borders)
    # items per workgroup: below 1, 1.2 (teams), 1.8 (pairs), 2.6 (teams of some jobs), 4.2 (none)
    for threads, workgroups, slice_ms in ((1024, 0, None), (1024, 0, 0.3), (512, 54, None), (1024, 35, 0.3),
                                          (512, 24, None), (256, 24, 0.3), (512, 15, None)):
        b.set_mapping(threads, workgroups)
        b.run(slice_ms)
        for r, (samples, H0, lat) in enumerate(refs):
            assert [tuple(map(int, s)) for s in zip(*b.samples(r))] == samples, (r, jobs[r], threads, workgroups)
            assert b.h0(r) == H0 and np.array_equal(b.get_lattice(r), lat), (r, jobs[r], threads, workgroups)
    b.free()


def test_served_large_and_small_together():
    # lattices of 4096^2 on several streams beside teams and one-workgroup jobs
    from paper_1110_6745_amd import okpz

    jobs = [(4096, 4096, 0.7, 0.1, 1, 25), (4096, 4096, 1.0, 0.0, 2, 40), (64, 64, 0.9, 0.0, 3, 200),
            (4096, 4096, 0.5, 0.5, 4, 12), (2048, 1024, 0.8, 0.0, 5, 60), (4096, 4096, 0.9, 0.0, 6, 31),
            (1024, 1024, 1.0, 0.0, 7, 50)]
    sv = okpz.Server(8 << 30)
    ids = [sv.submit(j) for j in jobs]
    sv.drain()
    for i, j in zip(ids, jobs):
        samples, H0, _ = alone(okpz, j, 0, 0.01)
        assert [tuple(map(int, s)) for s in zip(*sv.samples(i))] == samples, j
        assert sv.result(i)[1] == H0, j
    sv.free()
