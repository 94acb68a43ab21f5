"""The several-gates-per-sweep programs on the CPU: the planner's output
executed word by word in double precision against the gates applied one by
one (tests/tile_program.cpp), for random lists of every gate kind, with up to
three controls anywhere and matrices per row, on 4..14 qubits; both register
widths. Every LDS element is written once per round."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_19291_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("tile") / "tile_program")
    cmd = [hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", os.path.join(HERE, "tile_program.cpp"),
           os.path.join(CSRC, "tile.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("units", [0, 100000])      # four and three register bits
def test_programs_equal_the_gates(program, units):
    r = subprocess.run([program, "0", "200", str(units)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


def test_roundings_do_not_add_up_in_the_norm(program):
    """3000 matrices, rounded to FP32 one after the other, scale a state by no
    more than one rounding (2^-24) in all: one angle that by itself would
    drift, random rotations, general gates, phases, matrices per row."""
    r = subprocess.run([program, "norms"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
