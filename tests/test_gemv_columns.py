"""The column slices of the matrix-vector products (csrc/gemv_index.hpp), walked on
the CPU as the kernel walks them (tests/native/gemv_columns.cpp): for every block
size up to the largest one no load leaves the matrix, and every column is
multiplied once.  From 2048 columns on a slice can end in a stage of one to three
columns, fewer than the workgroup's waves."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_loads_stay_inside_the_matrix(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "gemv_columns")
    src = os.path.join(HERE, "native", "gemv_columns.cpp")
    subprocess.run([gxx, "-O2", "-std=c++17", src, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok 160 sizes\n", r.stdout + r.stderr
