"""CPU check of the mode products' loads: the offset arithmetic of csrc/modeslice.h, the one the kernel
uses, walked on the host over mode sizes 1 to 300, trailing sizes 1 to 40, both types and every tile
width; no vector may leave its input, and the vectors whose products are stored may not have moved.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_every_load_stays_in_its_buffer(tmp_path):
    exe = str(tmp_path / "mode_slices")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2309_03060_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "mode_slices.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
