"""CPU: the cuts of crowded intervals of output codes end and never leave their
stack, whatever the sampled products are.  The kernels' own header, compiled
for the host, against samples that an adversary picks: one code only, both
ends, one heavy code, products that crowd on every scale."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1004_4548_amd", "csrc")


def test_cuts_end_within_the_stack(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "interval_cuts")
    subprocess.run([cxx, "-O2", "-std=c++17", "-Wall", "-I", CSRC,
                    os.path.join(HERE, "interval_cuts.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
