"""The loss kernel's walk over half-faces (CPU build of the same header): whole, inside its range and ended, up to
the largest index a mesh may have, where a signed index would overflow in the step past the last batch."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_walk_at_the_largest_index(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "half_face_scan")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I",
                           os.path.join(ROOT, "paper_2002_08377_amd", "csrc"),
                           os.path.join(ROOT, "tests", "half_face_scan.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "half-face scan OK" in r.stdout, r.stdout + r.stderr
