"""The spectrum's scratch against its documented bytes, on the CPU (csrc/psd_plan.cpp is
plain C++), with the driver tests/c/psd_plan_check.cpp."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plans_stay_within_their_bytes(tmp_path):
    exe = str(tmp_path / "psd_plan_check")
    csrc = os.path.join(ROOT, "paper_1110_6745_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I", csrc,
                    os.path.join(csrc, "psd_plan.cpp"),
                    os.path.join(ROOT, "tests", "c", "psd_plan_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert (out.returncode, out.stdout.strip()) == (0, "psd plans ok"), out.stdout
