"""The plan builder's choice of kernels on the host (tests/check_plan_routes.cpp, linked with the builder)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_plan_routes(tmp_path):
    from paper_2606_15361_amd import build as B
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host g++")
    exe = str(tmp_path / "check_plan_routes")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I" + B.CSRC,
                    os.path.join(HERE, "check_plan_routes.cpp"), os.path.join(B.CSRC, "plan.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_table_shapes(tmp_path):
    from paper_2606_15361_amd import build as B
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host g++")
    exe = str(tmp_path / "check_table_shapes")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I" + B.CSRC,
                    os.path.join(HERE, "check_table_shapes.cpp"), os.path.join(B.CSRC, "plan.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
