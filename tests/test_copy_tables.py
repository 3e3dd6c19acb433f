"""The staged kernels' plan tables (copy chunks, offset words, parts), checked on the host against the
windows and inputs they stand for (tests/check_copy_tables.cpp, linked with the plan builder)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_copy_chunks_and_parts(tmp_path):
    from paper_2606_15361_amd import build as B
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host g++")
    exe = str(tmp_path / "check_copy_tables")
    subprocess.run([gxx, "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I" + B.CSRC,
                    os.path.join(HERE, "check_copy_tables.cpp"), os.path.join(B.CSRC, "plan.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
