"""Exact draws under memory limits and capture, by the library's own host code
with HIP's calls replaced (tests/shot_scratch.cpp, tests/fake_hip.h)."""

import os

import pytest

from tests import host_build


def test_draws_need_no_more_memory_than_without_the_sums(tmp_path):
    if not os.path.exists(host_build.HIPCC):
        pytest.skip("hipcc not found")
    host_build.run_with_library(str(tmp_path / "shot_scratch"), "shot_scratch.cpp")
