"""Host build of the order in which blocks take the points of a scan
(csrc/patch.hpp): every point once, the scan's row length found from its
points, and never more tiles per block than runs of points meet. CPU only."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PATCH = os.path.join(HERE, "..", "paper_2310_05766_amd", "csrc", "patch.hpp")


def test_patches_of_any_row_length(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = tmp_path / "patch_check"
    subprocess.run(["g++", "-O2", "-std=c++17", f'-DPATCH_HPP="{os.path.abspath(PATCH)}"', "-o", str(exe),
                    os.path.join(HERE, "host", "patch_check.cpp")], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "mismatches 0" in out.stdout
