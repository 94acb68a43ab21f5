"""C++ test programs linked with the library's objects (the regular build's, made
first if they are missing)."""

import glob
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2511_19291_amd")
HIPCC = "/opt/rocm/bin/hipcc"


def library_objects():
    srcs = [f for ext in ("hip", "cpp") for f in glob.glob(os.path.join(PKG, "csrc", "*." + ext))]
    objs = [os.path.join(PKG, "_build", os.path.basename(f) + ".o") for f in sorted(srcs)]
    if not all(os.path.exists(o) for o in objs):
        from paper_2511_19291_amd.csrc import build as hb
        hb.build()
    return objs


def build(exe, source, objs, *flags):
    cmd = [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", *flags, os.path.join(HERE, source), "-x", "none", *objs,
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def run_with_library(exe, source):
    """Build `source` with all of the library, without the HIP runtime (the
    program brings its own, tests/fake_hip.h), and run it."""
    build(exe, source, library_objects(), "-no-hip-rt")
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
