"""How the products with equal shares of the weight rows divide them (csrc/ring_share.h), walked on the host: integer
divisions by zero end the program there (without optimisation: a result that nobody uses counts too), where a GPU goes on
with whatever comes out."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_06282_amd", "csrc")


def test_every_group_comes_once(tmp_path):
    exe = str(tmp_path / "ring_share")
    subprocess.run(["g++", "-O0", "-std=c++17", "-I", CSRC, os.path.join(HERE, "ring_share.cpp"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.endswith("walks\n"), (r.returncode, r.stdout)
