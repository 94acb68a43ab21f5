"""The limit of dynamic LDS is one per kernel, not per launch: with a second
thread that launches a smaller program (or a second plan of narrower tiles) it
must not sink below what the first one launches with. tests/lds_limit.cpp,
linked with the library's kernels, records what they ask HIP for."""

import os
import subprocess

import pytest

from tests.test_sanitized_host import HIPCC, _device_objects

HERE = os.path.dirname(os.path.abspath(__file__))


def test_one_limit_per_kernel(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    objs = [o for o in _device_objects() if os.path.basename(o) in ("k_tile_adj.hip.o", "k_batch.hip.o")]
    exe = str(tmp_path / "lds_limit")
    cmd = [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", os.path.join(HERE, "lds_limit.cpp"), "-x", "none",
           *objs, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
