"""The segment lengths a row-streaming launch chooses from (paper_2405_12631_amd/csrc/wv_pieces.h)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_segment_length_once(tmp_path):
    """Each length that a number of segments gives, once, in the order of a search over all numbers, so that
    the first of the cheapest is the same; and few of them, since a launch makes the search."""
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    exe = str(tmp_path / "segments")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", os.path.join(HERE, "..", "paper_2405_12631_amd", "csrc"),
                    os.path.join(HERE, "segments_driver.cpp"), "-o", exe], check=True)
    for lo, hi in ((1, 600), (4095, 4097), (65535, 65536)):
        lines = subprocess.run([exe, str(lo), str(hi)], check=True, capture_output=True, text=True).stdout.splitlines()
        for h, line in zip(range(lo, hi + 1), lines):
            got = [int(v) for v in line.split()]
            assert got == sorted({-(-h // ns) for ns in range(1, h + 1)}, reverse=True), h
            assert len(got) <= 2 * h ** 0.5 + 1, h
