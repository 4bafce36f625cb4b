"""Index arithmetic and launch rules (csrc/host_rules.hpp) on the CPU, under
UndefinedBehaviorSanitizer (tests/host_rules/driver.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1405_0707_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_host_rules(tmp_path):
    exe = str(tmp_path / "host_rules")
    build = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=undefined",
             "-fno-sanitize-recover=all", "-I", CSRC,
             os.path.join(HERE, "host_rules", "driver.cpp"), "-o", exe]
    subprocess.run(build, check=True, capture_output=True, text=True, timeout=120)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(run.stdout)
    assert run.returncode == 0 and "ALL OK" in run.stdout, run.stdout + run.stderr
