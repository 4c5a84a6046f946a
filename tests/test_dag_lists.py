"""The task lists of launches over several blocks are merged from lists of single
blocks that the launches of a workspace share (csrc/dag.hpp, launch_list): the same
lists as a sort of all tasks (tests/native/dag_lists.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_merged_lists_equal_sorted_ones(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "dag_lists")
    src = os.path.join(HERE, "native", "dag_lists.cpp")
    subprocess.run([gxx, "-O2", "-std=c++17", src, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert (r.returncode, r.stdout) == (0, "ok 300 lists\n"), (r.returncode, r.stdout + r.stderr)
