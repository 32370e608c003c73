"""Workgroups that share weights are meant to run on one XCD, whose L2 then has them (csrc/xcd_grid.h): where they do not, only
the time of a call says so."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_06282_amd", "csrc")


def test_workgroups_of_a_place_run_on_one_xcd(tmp_path):
    exe = str(tmp_path / "xcd_grid")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, os.path.join(HERE, "xcd_grid.cpp"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
