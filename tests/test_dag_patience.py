"""The waits of the persistent diagonal-block launch are limited by time spent
polling (csrc/dag.hpp, Patience; tests/native/dag_patience.cpp): a process that is
held off the card for longer than the limit does not fail its evaluation."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_only_polling_counts(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "dag_patience")
    src = os.path.join(HERE, "native", "dag_patience.cpp")
    subprocess.run([gxx, "-O2", "-std=c++17", src, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout) == (0, "ok\n"), (r.returncode, r.stdout + r.stderr)
