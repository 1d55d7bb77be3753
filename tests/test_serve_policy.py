"""The serving policy's functions on the CPU (no GPU), beside the mock server of
the sanitized host checks."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_04857_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("serve") / "serve_checks")
    subprocess.check_call(["g++", "-O1", "-g", "-Wall", "-std=c++17", "-I", CSRC,
                           os.path.join(ROOT, "tests", "host", "serve_checks.cpp"),
                           os.path.join(CSRC, "serve_policy.cpp"), "-o", out])
    return out


@pytest.mark.parametrize("what", ["items", "blocks"])
def test_serve_policy(exe, what):
    p = subprocess.run([exe, what], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout + p.stderr
