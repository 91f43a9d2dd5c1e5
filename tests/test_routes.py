"""The dispatch rules between kernels (csrc/blas_sizes.h) against measured
times of both sides, on the host (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rules_take_the_faster_side(tmp_path):
    exe = str(tmp_path / "routes")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1512_04506_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "routes.cpp"), "-o", exe], check=True)
    p = subprocess.run([exe], capture_output=True, text=True)
    print(p.stdout)
    assert p.returncode == 0 and "FAIL" not in p.stdout, p.stdout
