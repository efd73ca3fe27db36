"""Packed task lists of the table kernel that leaves out the pairs beyond the
cutoff, checked by tests/near_pack_check.cpp over random item sets under
AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_packed_near_rule_invariants_under_sanitizers(tmp_path):
    exe = str(tmp_path / "near_pack_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1203_4037_amd", "csrc"),
                    os.path.join(ROOT, "tests", "near_pack_check.cpp"),
                    os.path.join(ROOT, "paper_1203_4037_amd", "csrc", "planner.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "near pack checks passed" in r.stdout, r.stdout + r.stderr
