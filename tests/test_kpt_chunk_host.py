"""Device memory of k-point grids, by the host code that sizes it: at most
256 MB of grids or one k-point's at a time, and where an allocation fails
half as many k-points down to one, which is what a solve needs at least."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_grid_chunks(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "kpt_chunk_check")
    r = subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                        os.path.join(HERE, "native", "kpt_chunk_check.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120).stdout
    rows = [line.split() for line in out.strip().splitlines()]
    chunk = {int(x): int(c) for k, x, c in (r[:3] for r in rows if r[0] == "chunk")}
    assert chunk == {1: 32, 17694720: 14, 255999999: 1, 256000001: 1, 5000000000: 1}
    fit = {int(r[1]): (int(r[2]), int(r[3])) for r in rows if r[0] == "fit"}
    assert fit == {1000: (32, 420), 420: (32, 420), 419: (16, 260), 200: (8, 180), 110: (1, 110), 109: (0, 110)}
