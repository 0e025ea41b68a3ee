"""The batch kernel's claim-word rules on the CPU (csrc/claim_word.h is plain C++ that
the kernel is built from), with the driver tests/c/claim_word_check.cpp."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_claim_words(tmp_path):
    exe = str(tmp_path / "claim_word_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I",
                    os.path.join(ROOT, "paper_1110_6745_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "claim_word_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert (out.returncode, out.stdout.strip()) == (0, "claim words ok"), out.stdout
