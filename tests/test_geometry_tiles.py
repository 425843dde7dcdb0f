"""The 8 x 32 preprocessing tiles' index functions, walked on the CPU
(tests/tile_check.cpp): every access inside its array, every cell staged, blurred
and owned once."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_small_tiles_cover_every_cell_once(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = tmp_path / "tile_check"
    b = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17",
                        "-I" + os.path.join(ROOT, "paper_1702_05156_amd", "csrc"),
                        os.path.join(ROOT, "tests", "tile_check.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, HIP_VISIBLE_DEVICES="-1"))
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout[-3000:]
