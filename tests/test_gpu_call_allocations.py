"""Calls that allocate nothing, neither device nor pinned host memory, from the first call of
a handle on: the HIP runtime's own log of API calls (a child process with
AMD_LOG_LEVEL=3) holds no allocation or release between two marks around the call.
"""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import os, sys
import numpy as np
from paper_1110_6745_amd import okpz

Lx, Ly = 320, 256
make = okpz.okpz_init if {copies} == 2 else okpz.okpz_init_in_place
other = make(Lx, Ly, 1.0, 0.0, 2)
other.sweep(2)
# the runtime's own first-use work is done by another handle
lat = other.get_lattice()
other.set_lattice(lat, 0, 0)
other.width(), other.w2(), other.psd_noalloc()
sim = make(Lx, Ly, 1.0, 0.0, 1)
sim.sweep(3)
batch = okpz.Batch([(64, 32, 1.0, 0.0, 1, 5)], 0.5)
batch.run()
os.write(2, b"\\nMARK begin\\n")
{call}
os.write(2, b"\\nMARK end\\n")
sim.free()
print("child ok", flush=True)
"""

CALLS = {
    "psd_noalloc": "sim.psd_noalloc()",
    "width": "sim.width()",
    "w2": "sim.w2()",
    "get_lattice": "sim.get_lattice()",
    "get_rows": "sim.get_rows(3, 5)",
    "set_lattice": "sim.set_lattice(lat, 0, 0)",
    "batch_get_lattice": "batch.get_lattice(0)",
}


@pytest.mark.parametrize("copies", [2, 1])
@pytest.mark.parametrize("call", list(CALLS))
def test_first_call_allocates_nothing(call, copies):
    env = dict(os.environ, AMD_LOG_LEVEL="3")
    r = subprocess.run([sys.executable, "-c", CHILD.format(call=CALLS[call], copies=copies)], cwd=ROOT, env=env,
                       capture_output=True, text=True, errors="replace", timeout=100)
    assert r.returncode == 0 and "child ok" in r.stdout, r.stderr[-2000:]
    log = r.stderr
    assert log.count("MARK begin") == 1 and log.count("MARK end") == 1
    during = log[log.index("MARK begin"):log.index("MARK end")]
    assert re.search(r"hip(StreamSynchronize|Memcpy)", during), "the runtime's log holds no calls"
    found = re.findall(r"hip\w*(?:Malloc|HostAlloc|HostRegister|Free)\w* *\(", during)
    assert not found, found
    assert re.search(r"hipMalloc *\(", log), "the log would not show an allocation"


def test_measurements_of_many_handles():
    # more handles than one pinned slab serves, freed and made again in between
    import oracle
    from paper_1110_6745_amd import okpz

    Lx, Ly = 64, 32

    def made(seed):
        sim = okpz.okpz_init(Lx, Ly, 0.9, 0.2, seed)
        sim.sweep(1 + seed % 3)
        return sim

    def want(seed):
        lat = oracle.flat(Lx, Ly)
        return oracle.width_sums(lat, oracle.run(lat, 0.9, 0.2, seed, 0, 1 + seed % 3, 0))

    sims = {seed: made(seed) for seed in range(130)}
    for seed in range(0, 130, 2):
        sims.pop(seed).free()
    sims.update({seed: made(seed) for seed in range(200, 240)})
    for seed, sim in sims.items():
        assert sim.width() == want(seed), seed
    for sim in sims.values():
        sim.free()


def test_transfers_and_spectra_of_several_threads():
    # all of them use the GPU's one scratch, in turns
    import threading

    import numpy as np

    from paper_1110_6745_amd import okpz
    from tests import inputs

    sizes = [(4096, 4096), (320, 4096), (8192, 2080), (96, 64)]
    lats = [inputs.separable_rows(inputs.balanced_bits(Lx, i), inputs.balanced_bits(Ly, i + 9), 0, Ly)
            for i, (Lx, Ly) in enumerate(sizes)]
    sims = [okpz.okpz_init(Lx, Ly, 1.0, 0.0, 1) for Lx, Ly in sizes]
    spectra, wrong = [], []
    for sim, lat in zip(sims, lats):
        sim.set_lattice(lat, 0, 0)
        spectra.append(sim.psd())

    def work(i):
        for _ in range(4):
            sims[i].set_lattice(lats[i], 2 * i, 1)
            if not np.array_equal(sims[i].get_lattice(), lats[i]):
                wrong.append((sizes[i], "lattice"))
            if not all(np.array_equal(a, b) for a, b in zip(sims[i].psd_noalloc(), spectra[i])):
                wrong.append((sizes[i], "spectrum"))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not any(t.is_alive() for t in threads)
    assert not wrong, wrong
    for sim in sims:
        sim.free()


def test_batch_memory():
    # two copies of each lattice (16 bytes per row of 32 sites), and little else
    import torch

    from paper_1110_6745_amd import okpz

    n, Ly = 2000, 8192
    torch.cuda.init()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    batch = okpz.Batch([(32, Ly, 1.0, 0.0, i, 1) for i in range(n)], 0.5)
    used = free - torch.cuda.mem_get_info()[0]
    copies = n * 16 * Ly
    assert used <= copies + n * 1024 + (4 << 20), (used, copies)
    batch.free()
