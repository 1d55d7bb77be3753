"""The memory that a thread keeps between its lone solves, against a test
double of the HIP calls it makes (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_04857_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("workspace") / "workspace_checks")
    subprocess.check_call(["g++", "-O1", "-g", "-Wall", "-std=c++17", "-pthread",
                           "-I", os.path.join(HOST, "fakehip"), "-I", CSRC,
                           os.path.join(HOST, "workspace_checks.cpp"),
                           os.path.join(CSRC, "workspace.cpp"), "-o", out])
    return out


@pytest.mark.parametrize("what", ["capture", "devices", "waits", "fork"])
def test_workspace(exe, what):
    p = subprocess.run([exe, what], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout + p.stderr
