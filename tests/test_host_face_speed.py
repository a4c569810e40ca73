"""The face speed of PLM stage 2 in FP64 (CPU build of the same header): along an antipode as exact as along its
direction."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_antipode_is_as_exact_as_its_direction(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "face_speed")
    subprocess.check_call(["g++", "-std=gnu++17", "-O2", "-ffp-contract=off", "-I",
                           os.path.join(ROOT, "paper_2002_08377_amd", "csrc"),
                           os.path.join(ROOT, "tests", "face_speed.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "face speed OK" in r.stdout, r.stdout + r.stderr
