"""The solve's tables checked on the host (no GPU; tests/solve_check.cpp, built
here with the host compiler): which sizes run the recursion in steps, the
least-squares samples by pair, and the step schedule at every radius."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1701_00581_amd", "csrc")


def _run(tmp_path, source, cases):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", source),
                    os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe, *cases], check=True, capture_output=True, text=True)
    lines = r.stdout.strip().splitlines()
    assert len(lines) == len(cases)
    return lines


def test_steps_only_where_no_number_of_patches_is_slower(tmp_path):
    """Where steps win for few patches and lose past one round of workgroups
    (N = 128 but for R = 10 at a high cut-off; N = 64 with three or more pairs
    per lane), and where the cut-off is close to R, the recursion runs in
    units."""
    steps = ["64:31:1", "64:31:4", "64:31:6", "64:12:5", "64:6:3", "128:63:10", "128:60:10"]
    units = ["64:31:7", "64:31:8", "64:31:10", "64:31:12", "64:31:13", "64:16:15", "64:12:10", "64:4:2", "64:2:1",
             "128:63:1", "128:63:6", "128:63:9", "128:63:11", "128:63:12", "128:63:16", "128:59:10", "128:30:10",
             "128:12:10", "128:3:2"]
    for line in _run(tmp_path, "solve_check.cpp", steps + units):
        assert f" in_steps={int(line.split()[0] in steps)} " in line, line


def test_least_squares_pairs_hold_every_sample_once(tmp_path):
    cases = [f"64:31:{R}" for R in range(1, 13)] + ["128:63:10", "128:63:12", "64:13:12", "64:5:4", "64:2:1"]
    for line in _run(tmp_path, "solve_check.cpp", cases + ["64:31:13"]):
        none = line.startswith("64:31:13 ")
        assert line.endswith(" bad=0") and (" pairs=0 " in line) == none, line


def test_step_schedule_at_every_radius(tmp_path):
    for line in _run(tmp_path, "phase_check.cpp", [f"{N}:{uc}:{R}" for N, uc in ((64, 31), (128, 63))
                                                   for R in range(1, 13)]):
        assert line.endswith(" bad=0") and " steps=0 " not in line, line
