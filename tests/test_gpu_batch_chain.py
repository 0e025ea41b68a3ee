"""Jobs of one item per sweep, which a workgroup advances several sweeps per claim,
mixed with jobs of many items, against the same jobs run alone: more and fewer jobs
than workgroups, lengths around the sweeps of one claim (32), samples at every sweep
of a claim, both thread-cell borders, slices that stop inside a claim, and one claim
policy each (items per workgroup below 2.5, below 4, and more).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def alone(okpz, job, borders, m):
    Lx, Ly, p, q, seed, t_max = job
    sim = okpz.okpz_init(Lx, Ly, p, q, seed)
    sim.set_cell_borders(borders)
    out = []
    for t in okpz.sampling_times(t_max, m):
        out.append((t, *sim.width(t)))
    sim.sweep(t_max - sim.time())
    res = out, sim.h0(), sim.get_lattice()
    sim.free()
    return res


def jobs_of(p, q):
    # 1 item: up to 256 x 256; 2 to 16 items: the rest
    sizes = [(32, 32), (64, 32), (96, 96), (256, 256), (160, 224), (32, 2048), (32, 2080), (512, 256), (1024, 512),
             (992, 96)]
    lengths = [0, 1, 31, 32, 33, 64, 65, 97]
    return [(Lx, Ly, p, q, 7 * i + 1, lengths[(i + k) % len(lengths)])
            for k in range(2) for i, (Lx, Ly) in enumerate(sizes)]


@pytest.mark.parametrize("p,q,borders", [(1.0, 0.0, 0), (0.8, 0.1, 0), (1.0, 0.0, 1)])
@pytest.mark.parametrize("threads,workgroups", [(1024, 0), (512, 7), (256, 3)])
def test_chained_and_claimed_jobs(p, q, borders, threads, workgroups):
    from paper_1110_6745_amd import okpz

    jobs, m = jobs_of(p, q), 0.02
    b = okpz.Batch(jobs, m)
    b.set_cell_borders(borders)
    b.set_mapping(threads, workgroups)
    refs = [alone(okpz, j, borders, m) for j in jobs]
    for slice_ms in (None, 0.2):
        b.run(slice_ms)
        for r, (samples, H0, lat) in enumerate(refs):
            assert [tuple(map(int, s)) for s in zip(*b.samples(r))] == samples, (r, jobs[r], slice_ms)
            assert b.h0(r) == H0 and np.array_equal(b.get_lattice(r), lat), (r, jobs[r], slice_ms)
    b.free()


def test_width_of_long_and_narrow_jobs():
    # rows of 1 to 64 words side by side in a wavefront, and longer rows
    from paper_1110_6745_amd import okpz

    jobs = [(Lx, Ly, 0.9, 0.2, 3 + i, 12) for i, (Lx, Ly) in enumerate(
        [(32, 64), (64, 96), (96, 32), (160, 64), (288, 96), (544, 32), (1056, 64), (2048, 32), (2080, 64),
         (4128, 32), (8192, 64)])]
    b = okpz.Batch(jobs, 0.3)
    b.run()
    for r, j in enumerate(jobs):
        samples, H0, lat = alone(okpz, j, 0, 0.3)
        assert [tuple(map(int, s)) for s in zip(*b.samples(r))] == samples, j
        assert b.h0(r) == H0 and np.array_equal(b.get_lattice(r), lat), j
    b.free()
