"""The waits of the kernel of 256 query rows per workgroup (csrc/tva_wide.hip), on the host: its loop over the tiles and the
merge of its pieces are templates that the kernel and this test walk with steps of their own (csrc/tva_wide_order.h).  A run
on the card says nothing about a wait that is missing, because the transfer has nearly always arrived by then."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_06282_amd", "csrc")


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("wide_order") / "wide_order")
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-pthread", "-I", CSRC, os.path.join(HERE, "wide_order.cpp"), "-o", exe],
                   check=True, timeout=120)
    return lambda what: subprocess.run([exe, what], capture_output=True, text=True, timeout=300)


def test_every_tile_read_was_waited_for(walk):
    """Every piece of up to 100 tiles without masks and up to 6 with, both head dimensions."""
    r = walk("tiles")
    assert r.returncode == 0, r.stdout[-4000:]


def test_a_merge_is_complete_whoever_is_held_up(walk):
    """Up to nine pieces, in orders drawn at random, with waits that end at once, soon, or practically never; the first to
    come has to go on in some (its partner stopped waiting and left its results before it did)."""
    r = walk("pieces")
    assert r.returncode == 0, r.stdout[-4000:]
