"""The phase recursion's step schedule checked on the host (no GPU): every
sample summed once, from phasors that are known by then
(tests/phase_check.cpp, built here with the host compiler)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1701_00581_amd", "csrc")


def test_phase_steps_cover_every_sample_once(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "phase_check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "phase_check.cpp"),
                    os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True, capture_output=True)
    cases = ["128:63:12", "128:63:10", "128:63:9", "128:63:1", "128:20:12", "128:3:2", "64:31:12", "64:31:8",
             "64:31:11", "64:2:1", "64:5:4"]
    r = subprocess.run([exe, *cases, "128:63:13"], check=True, capture_output=True, text=True)
    lines = r.stdout.strip().splitlines()
    assert len(lines) == len(cases) + 1
    for line in lines[:-1]:
        assert line.endswith(" bad=0") and " steps=0 " not in line, line
    assert " steps=0 " in lines[-1], lines[-1]      # too many pairs: no step schedule
