"""The waits of the kernel of 256 query rows per workgroup (csrc/tva_wide.hip), on the host: its loop over the tiles is a
template that the kernel and this test walk with steps of their own (csrc/tva_wide_order.h).  A run on the card says nothing
about a wait that is missing, because the transfer has nearly always arrived by then."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_06282_amd", "csrc")


def test_every_tile_read_was_waited_for(tmp_path):
    """Every piece of up to 100 tiles without masks and up to 6 with, both head dimensions."""
    exe = str(tmp_path / "wide_order")
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-I", CSRC, os.path.join(HERE, "wide_order.cpp"), "-o", exe], check=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
