"""The joined task lists of the persistent diagonal-block factorisation
(csrc/dag.hpp, join), emulated on the CPU (tests/native/dag_joined.cpp): no task
lost, waits only on earlier tasks, no deadlock with 1 to 256 workers, no
conflicting tasks runnable together, and the result of a plain Cholesky and
inversion, for 1 to 18 tiles (groups of four and eight with remainders)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_joined_task_lists_emulated(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "dag_joined")
    src = os.path.join(HERE, "native", "dag_joined.cpp")
    subprocess.run([gxx, "-O2", "-std=c++17", src, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.count("ok joined") == 9 * 3 * 3 * 2
