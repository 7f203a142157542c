"""The staged operations' LDS layout (csrc/pbz_stage_layout.h), compiled for the CPU and checked for every kept count and index
size: sizes, limits, and the 16-byte alignment that their vector accesses need."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_layouts_of_every_kept_count(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "stage_layout_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2406_11209_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "stage_layout_check.cpp"), "-o", exe], check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True).stdout
    assert out.startswith("ok"), out
