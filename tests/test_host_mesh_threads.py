"""The host half of the mesh upload on a team of threads (CPU): the same index, orders, staging sizes and
refusals as a serial recomputation, on a mesh large enough for the team and with the last group of cells
partly filled."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_threaded_upload_matches_serial(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "host_mesh_threads")
    src = os.path.join(ROOT, "tests", "host_mesh_threads.cpp")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-I",
                           os.path.join(ROOT, "paper_2002_08377_amd", "csrc"), src, "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "host mesh threads OK" in r.stdout, r.stdout + r.stderr
