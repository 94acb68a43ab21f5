"""n_sweeps of the fusion autotuner's choices against the launches of the library's
own host code, HIP's calls replaced (tests/sweep_counts.cpp, tests/fake_hip.h)."""

import os

import pytest

from tests import host_build


def test_n_sweeps_counts_passes(tmp_path):
    if not os.path.exists(host_build.HIPCC):
        pytest.skip("hipcc not found")
    host_build.run_with_library(str(tmp_path / "sweep_counts"), "sweep_counts.cpp")
