"""Exact draws under memory limits and capture, by the library's own host code
with HIP's calls replaced (tests/shot_scratch.cpp, tests/fake_hip.h)."""

import glob
import os
import subprocess

import pytest

from tests.test_sanitized_host import HIPCC, ROOT, _device_objects

HERE = os.path.dirname(os.path.abspath(__file__))


def build_with_library(exe, source):
    """Compile `source` and link it with the library's objects, not with HIP."""
    _device_objects()
    objs = sorted(glob.glob(os.path.join(ROOT, "paper_2511_19291_amd", "_build", "*.o")))
    cmd = [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-no-hip-rt", os.path.join(HERE, source), "-x", "none",
           *objs, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_draws_need_no_more_memory_than_without_the_sums(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "shot_scratch")
    build_with_library(exe, "shot_scratch.cpp")
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
