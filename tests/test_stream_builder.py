"""The stream encoding's host builder (CPU only): the encoding of matrices at
the sizes where it can go wrong is walked as the kernels walk it -- every
pixel once, no two lanes of one LDS access in one element, every bin's
partial sums in its list -- under AddressSanitizer and
UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

from tests.helpers import ROOT

CSRC = os.path.join(ROOT, "paper_1412_6367_amd", "csrc")

CASES = [
    # h, w, center_y, center_x, npt, npt_azim, unit, split, tile_px (, range): tiles expected
    (1, 1, 0.5, 0.5, 4, 0, 0, 1, 1024),               # under four pixels: refused
    (1, 4, 0.5, 2.5, 3, 0, 0, 1, 1024),               # the smallest
    (2, 2, 1.0, 1.0, 2, 0, 0, 1, 1024),
    (1, 17, 0.5, 8.5, 5, 0, 0, 1, 1024),              # one row
    (300, 1, 3.5, 0.5, 40, 0, 0, 1, 1024),            # one column
    (37, 63, 10.25, 40.5, 61, 0, 0, 1, 1024),         # one strip, ragged
    (64, 64, 32.0, 32.0, 64, 0, 0, 1, 1024),          # whole blocks
    (65, 65, 32.5, 32.5, 64, 0, 0, 1, 1024),          # one pixel more, two strips
    (33, 129, -5.0, 70.0, 40, 0, 0, 1, 1024),         # beam off the detector
    (31, 29, 15.5, 14.5, 300, 0, 0, 1, 1024),         # bins finer than pixels
    (40, 40, 20.0, 20.0, 4000, 0, 0, 1, 1024),        # over 63 bins a pixel: refused
    (200, 200, 100.0, 100.0, 3000, 0, 0, 1, 1024),    # tiles halved to a few pixels: refused
    (200, 200, 100.0, 100.0, 1200, 0, 0, 1, 1024),    # windows that halve the tiles
    (300, 280, 150.2, 139.7, 1, 0, 0, 1, 1024),       # one bin
    (300, 280, 150.2, 139.7, 7, 0, 0, 1, 3072),       # a few bins: 64 copies
    (50, 60, 25.0, 30.0, 37, 0, 0, 1, 1024, 5e-4, 2.5e-3),   # pixels that feed no bin
    (200, 260, 100.0, 130.0, 37, 0, 0, 1, 1024, 5e-4, 2e-3),  # tiles that feed no bin
    (50, 60, 25.3, 30.7, 37, 0, 0, 0, 1024),          # no split
    (141, 138, 20.6, 18.2, 150, 0, 4, 2, 2048),       # full split in q
    (260, 250, 130.0, 125.0, 200, 0, 3, 1, 3072),
    (150, 140, 70.3, 75.8, 20, 12, 0, 1, 1024),       # radius x azimuth
    (150, 141, 75.0, 70.5, 30, 90, 0, 1, 1024),       # the beam on a pixel's edge
    (151, 141, 75.5, 70.5, 8, 720, 0, 1, 1024),       # few entries a partial sum: refused
    (601, 601, 300.5, 300.5, 4, 720, 0, 1, 1024),     # in a pixel of more runs than a window holds
    (130, 60, -40.0, 30.0, 25, 36, 4, 1, 2048),       # beam off the detector
    (120, 120, 61.2, 58.9, 15, 24, 0, 2, 1024),       # full split
    (100, 90, 50.5, 44.5, 12, 16, 0, 0, 1024),        # no split
    (60, 60, 30.0, 30.0, 60, 360, 0, 1, 1024),        # bins finer than pixels: refused
    (600, 500, 301.3, 249.1, 100, 90, 0, 1, 2048),    # several threads
]


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("stream") / "stream_harness")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off",
                        "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        os.path.join(CSRC, "plan_builder.cpp"),
                        os.path.join(CSRC, "stream_builder.cpp"),
                        os.path.join(ROOT, "tests", "sanitize", "stream_harness.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_stream_encoding(case, harness):
    r = subprocess.run([harness, *map(str, case)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    refused = case[0] * case[1] < 4 or case[4] in (3000, 4000) or case[4:6] in ((60, 360), (8, 720))
    assert (r.stdout.strip() == "refused") == refused, r.stdout
