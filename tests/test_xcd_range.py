"""How the blocks of a grid share a list of bricks, tiles or segments: compiled for the host, over
every grid of up to 64 blocks and lists from empty to some rounds."""
import os
import subprocess

import pytest

from tests.cpu_hip import emu

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "cpu_hip")
pytestmark = pytest.mark.skipif(not os.path.exists(emu.CLANG), reason="no host clang++")


def test_every_entry_once_and_no_extra_round(tmp_path):
    exe = str(tmp_path / "xcd_range_check")
    subprocess.check_call([emu.CLANG, "-std=c++20", "-O2", "-Wno-unknown-attributes", "-I", HERE,
                           "-I", os.path.join(emu.ROOT, "include"), "-I", emu.CSRC, "-x", "c++",
                           os.path.join(HERE, "xcd_range_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
