"""The rotation log of the one-workgroup subspace step holds what its kernels
may write: csrc/kernels_sub.hip compiled for the host with the launches
recorded, at every band count and at sweep limits beyond the log's size (the
tuning key SGO_RR_SWEEPS takes any positive number)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_sweeps_fit_the_rotation_log(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "sub_launch_check")
    r = subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        os.path.join(HERE, "native", "sub_launch_check.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120).stdout
    rows = [[int(x) for x in line.split()] for line in out.strip().splitlines()]
    assert len(rows) == (198 - 32) * 7
    for n, asked, sweeps, rotations, room in rows:
        assert sweeps >= min(asked, 40), "n=%d: %d sweeps of %d" % (n, sweeps, asked)
        assert rotations <= room, "n=%d: %d sweeps asked, %d rotations, room for %d" % (n, asked, rotations, room)
