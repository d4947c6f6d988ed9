"""The tile sequence of a launch, and of the rest that a block of whole tiles
leaves (tests/tile_regions_check.cpp), on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_every_tile_once_and_no_division_by_zero(tmp_path):
    exe = str(tmp_path / "tile_regions_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I" + os.path.join(ROOT, "paper_2506_11209_amd", "csrc"),
                    os.path.join(ROOT, "tests", "tile_regions_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
