"""The rule by which launches reserve LDS to cap their occupancy (host code), on
the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not found")
def test_reservations_fit_one_workgroup(tmp_path):
    exe = tmp_path / "lds_reservation_check"
    subprocess.run(["hipcc", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2510_26709_amd", "csrc"),
                    os.path.join(ROOT, "tests", "lds_reservation_check.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
