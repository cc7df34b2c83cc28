"""The static entry point's choice among its plans (host code), on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_2510_26709_amd")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not found")
def test_kind_of_the_plan_near_the_scratch_limit(tmp_path):
    exe = tmp_path / "plan_kind_check"
    subprocess.run(["hipcc", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(LIB_DIR, "csrc"), os.path.join(ROOT, "tests", "plan_kind_check.cpp"),
                    f"-L{LIB_DIR}", "-l:libarctopk.so", f"-Wl,-rpath,{LIB_DIR}", "-o", str(exe)],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
