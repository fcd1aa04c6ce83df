"""The rules that choose between launches (csrc/route.cpp), on the CPU: each
agrees with the measured times on the grids that its comment names."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2011_02600_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_route_rules(tmp_path):
    exe = str(tmp_path / "route_check")
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, os.path.join(HERE, "host", "route_check.cpp"),
           os.path.join(CSRC, "route.cpp"), os.path.join(CSRC, "tile_shape.cpp"), "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout
