"""n_sweeps of the fusion autotuner's choices against the launches of the library's
own host code, HIP's calls replaced (tests/sweep_counts.cpp, tests/fake_hip.h)."""

import os
import subprocess

import pytest

from tests.test_sanitized_host import HIPCC
from tests.test_shot_scratch import build_with_library


def test_n_sweeps_counts_passes(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "sweep_counts")
    build_with_library(exe, "sweep_counts.cpp")
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
