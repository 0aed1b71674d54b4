"""How the MLP kernels cut their work (csrc/mlp_plan.h): the header itself, compiled
with g++ and walked on the CPU (tests/c/mlp_plan.cpp)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_mlp_plan(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "mlp_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I",
                    os.path.join(ROOT, "paper_2211_00889_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "c", "mlp_plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-2000:]
