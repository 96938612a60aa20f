"""The cut of the gridding rows into runs and chunks and the rule of the default chunk size
(grid_cut.hpp) on the CPU, built with g++ under AddressSanitizer + UndefinedBehaviorSanitizer: the
bounds hold for the chunks as they are cut, for windows whose runs fill chunks badly, at the bounds
themselves and for random tiles; 256 and 512 are taken as asked for.  psara_footprint counts the
slots that the default size may be cut to."""
import os
import shutil
import subprocess

import pytest

from paper_1801_02417_amd import psara as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_chunks_keep_the_bounds_as_cut(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "grid_cut")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_1801_02417_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "grid_cut.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "windows of 33: 128 entries" in r.stdout


def test_footprint_counts_the_smallest_chunks():
    """4096 rows spread evenly over the 16 gridding tiles of a 32^2 image are cut into chunks of 64: 64
    partial slots.  Their number in the footprint, from the footprints at eight and four taps, which
    differ by the size of a slot, 23 x 23 against 19 x 19 cells of 64 bytes (and by under half a
    slot's difference in the row lists)."""
    eight, four = (P.psara_footprint(32, 4096, taps, 3, P.ALL_BASES, P.PSARA_FP64) for taps in (8, 4))
    assert (eight - four) // ((23 * 23 - 19 * 19) * 64) >= 64
