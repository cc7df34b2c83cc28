"""The projection's vectorised Box-Muller (host code) against its definition
through the C library's log, cos and sqrt: the same bits, and an error well
inside the margin that sends a value to the definition, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_26709_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not found")
@pytest.mark.parametrize("opt", ["-O1", "-O3"])
def test_projection_values_have_the_definitions_bits(tmp_path, opt):
    exe = tmp_path / "projection_values_check"
    cmd = ["hipcc", "-std=c++17", opt, "-ffp-contract=off", "-fno-fast-math", "-fno-math-errno",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "projection_values_check.cpp"), "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe), "100000"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("ok"), r.stdout
