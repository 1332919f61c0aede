"""The cut of the tile line, computed on the host by the functions that the kernels use (plan_host.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_a_cut_covers_the_line_once_whatever_the_history_holds(tmp_path):
    exe = str(tmp_path / "plan_host")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-o", exe, os.path.join(HERE, "plan_host.cpp")], check=True)
    got = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert got.returncode == 0, got.stdout
