"""The limit of dynamic LDS is one per kernel, not per launch: with a second
thread that launches a smaller program (or a second plan of narrower tiles) it
must not sink below what the first one launches with. tests/lds_limit.cpp,
linked with the library's kernels, records what they ask HIP for."""

import os
import subprocess

import pytest

from tests import host_build


def test_one_limit_per_kernel(tmp_path):
    if not os.path.exists(host_build.HIPCC):
        pytest.skip("hipcc not found")
    objs = [o for o in host_build.library_objects() if os.path.basename(o) in ("k_tile_adj.hip.o", "k_batch.hip.o")]
    exe = str(tmp_path / "lds_limit")
    host_build.build(exe, "lds_limit.cpp", objs)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
