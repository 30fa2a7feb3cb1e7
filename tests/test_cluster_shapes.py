"""Shapes of cluster solves (host arithmetic): within LDS and the literal fields at
every size, and one kernel per launch whatever a batch brings together."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2402_03640_amd", "csrc")


def test_cluster_shapes(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs a host compiler")
    exe = str(tmp_path / "shapes")
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, os.path.join(HERE, "cluster_shapes.cpp"),
                    "-o", exe], check=True)
    run = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
    assert run.stdout.startswith("ok "), run.stdout
