"""Registers of the single-workgroup sweep kernels (no GPU needed): they advance every
lattice of up to 1024 cells in all acceptance modes and both cell borders, bound by the
chain of their steps, so none may spill to scratch.  One 1024-thread workgroup per CU is
enough for them (a launch is one workgroup), so unlike the other 1024-thread kernels
they are not held to 80 scalar registers.
"""
import json
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RESOURCES = os.path.join(ROOT, "paper_1110_6745_amd", "_build", "kernel_resources.json")


def test_chain_kernels_do_not_spill():
    if not os.path.exists(RESOURCES):
        pytest.skip("no kernel resource record: run build() first")
    with open(RESOURCES) as f:
        kernels = {n: r for n, r in json.load(f).items() if "sweep_chain_kernel" in n}
    modes = {re.search(r"ILi(\d+)ELi(\d+)ELb(\d)E", n).groups() for n in kernels}
    # growth, fixed and drawn acceptance, each with dead (0) and delayed (4) cell borders;
    # one 256 x 256 block, or smaller ones with a block or lane origin per wave
    assert modes == {(str(m + c), b, l) for m in range(3) for c in (0, 4)
                     for b, l in (("256", "0"), ("0", "0"), ("0", "1"))}
    for n, r in kernels.items():
        assert r["scratch"] == 0, (n, r)
        assert r["occupancy"] >= 4, (n, r)  # 16 waves of one workgroup on four SIMDs
        assert r["lds"] <= 160 * 1024, (n, r)
