"""The multigroup step takes the faster of two measured forms (CPU build of the rule)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rule_takes_the_faster_form(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "mg_rule")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2002_08377_amd", "csrc"),
                           os.path.join(ROOT, "tests", "mg_rule.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "multigroup rule OK" in r.stdout, r.stdout + r.stderr
