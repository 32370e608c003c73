"""The words of a workspace's header through which the workgroups of a call meet (csrc/jk_words.h): the protocols of the
kernels that use them take turns on one header, on the host."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_06282_amd", "csrc")


def test_calls_of_every_kind_take_turns_on_one_header(tmp_path):
    """Sixty calls on each of forty headers, in orders drawn at random: a call that counts in a word that another kind of call
    leaves something in never merges, or merges too early."""
    exe = str(tmp_path / "header_words")
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-pthread", "-I", CSRC, os.path.join(HERE, "header_words.cpp"), "-o", exe],
                   check=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
