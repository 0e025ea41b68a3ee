"""Results of a batch read at every stage of its life (before a run, between slices,
after a run, after a second run and after an autotuning), and a batch whose results
exceed the size that a run copies to the host at once (64 MiB).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def results(b, jobs):
    return [(tuple(map(tuple, b.samples(r))), b.h0(r)) for r in range(jobs)]


def test_results_at_every_stage():
    from paper_1110_6745_amd import okpz

    jobs = [(64, 96, 1.0, 0.0, 5, 40), (256, 256, 0.9, 0.3, 6, 25), (512, 1024, 1.0, 0.0, 7, 300), (32, 32, 1.0, 0.0, 8, 0)]
    alone = []
    for Lx, Ly, p, q, seed, t in jobs:
        sim = okpz.okpz_init(Lx, Ly, p, q, seed)
        sim.sweep(t)
        alone.append(sim.h0())
        sim.free()
    b = okpz.Batch(jobs, 0.05)
    with pytest.raises(okpz.OkpzError):
        b.samples(0)
    b.run()
    first = results(b, len(jobs))
    assert [h for _, h in first] == alone
    stage = []
    b.run(0.5, lambda done: stage.append((done, b.h0(2))))  # between slices: the state on the device
    assert stage[0][0] < len(jobs) and stage[-1][1] == alone[2]
    assert all(x[1] <= y[1] for x, y in zip(stage, stage[1:])) and stage[0][1] < alone[2]
    assert results(b, len(jobs)) == first
    b.autotune(8)
    with pytest.raises(okpz.OkpzError):
        b.samples(0)
    assert b.h0(2) < alone[2]  # of the trial sweeps
    b.run()
    assert results(b, len(jobs)) == first
    b.free()


def test_results_beyond_the_host_copy():
    from paper_1110_6745_amd import okpz

    t, n = 27000, 560  # a sample every ten sweeps: 560 x 2700 of 48 bytes
    jobs = [(32, 32, 1.0, 0.0, i + 1, t) for i in range(n)]
    big = okpz.Batch(jobs, 1e-6)
    big.run()
    few = okpz.Batch([jobs[0], jobs[117], jobs[n - 1]], 1e-6)
    few.run()
    assert n * len(okpz.sampling_times(t, 1e-6)) * 48 > 64 << 20
    for i, r in enumerate((0, 117, n - 1)):
        a, c = big.samples(r), few.samples(i)
        assert a[0][-1] == t and all(np.array_equal(x, y) for x, y in zip(a, c))
        assert big.h0(r) == few.h0(i)
    big.free()
    few.free()
