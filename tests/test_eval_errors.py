"""Every launch of a PaiNN evaluation that fails is reported (CPU only: the
launches are stubs, tests/host/eval_errors.cpp)."""
import os
import shutil
import subprocess

import pytest

from paper_2506_04055_amd import build as B

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host", "eval_errors.cpp")


def test_failed_launches_are_reported(tmp_path):
    if not shutil.which(B.HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "eval_errors")
    r = subprocess.run([B.HIPCC, "-x", "hip", *B.CFLAGS, "-O0", SRC, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
