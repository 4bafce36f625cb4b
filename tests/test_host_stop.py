"""The host eigensolvers of the restart end early when the thread that started
them asks for it (csrc/eig_host.hpp, StopToken; tests/host_stop/driver.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1405_0707_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_eigensolvers_stop(tmp_path):
    exe = str(tmp_path / "host_stop")
    build = ["g++", "-std=c++17", "-O2", "-pthread", "-I", CSRC,
             os.path.join(HERE, "host_stop", "driver.cpp"),
             os.path.join(CSRC, "eig_host.cpp"), "-o", exe]
    subprocess.run(build, check=True, capture_output=True, text=True, timeout=120)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(run.stdout)
    assert run.returncode == 0 and "ALL OK" in run.stdout, run.stdout + run.stderr
