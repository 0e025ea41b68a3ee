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
other.width(), other.w2(), other.psd_noalloc()  # the runtime's own first-use work is done by another handle
sim = make(Lx, Ly, 1.0, 0.0, 1)
sim.sweep(3)
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
