"""Which plans may walk on wide words, by the planner on the CPU (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_04857_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def test_wide_plans(tmp_path):
    exe = str(tmp_path / "plan_checks")
    subprocess.check_call(["g++", "-O1", "-g", "-Wall", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, os.path.join(ROOT, "tests", "host", "plan_checks.cpp"),
                           os.path.join(CSRC, "plan.cpp"), "-o", exe])
    p = subprocess.run([exe, "wide"], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout + p.stderr
