"""The preprocessing kernels' index functions on every tile they are compiled for,
walked on the CPU (tests/tile_walk.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_every_tile_covers_every_cell_once(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = tmp_path / "tile_walk"
    b = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17",
                        "-I" + os.path.join(ROOT, "paper_1702_05156_amd", "csrc"),
                        os.path.join(ROOT, "tests", "tile_walk.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, HIP_VISIBLE_DEVICES="-1"))
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout[-3000:]
