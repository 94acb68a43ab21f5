"""Rules of the several-gates-per-sweep path that hold without a GPU
(tests/tile_rules.cpp, linked with the planner)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_19291_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("tile") / "tile_rules")
    cmd = [hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", os.path.join(HERE, "tile_rules.cpp"),
           os.path.join(CSRC, "tile.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(name):
        r = subprocess.run([exe, name], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout

    return run


def test_programs_are_aligned(rules):
    rules("layout")


def test_lone_gates_keep_the_lists_matrices(rules):
    rules("single")


def test_short_lists_take_the_faster_sweeps(rules):
    rules("short")


def test_few_strings_on_many_rows_go_by_x(rules):
    rules("strings")
