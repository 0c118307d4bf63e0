"""Images whose positions do not fit the stream kernels' 32 bits keep their
stored layout (CPU only)."""
import os
import shutil
import subprocess

import pytest

from tests.helpers import ROOT

CSRC = os.path.join(ROOT, "paper_1412_6367_amd", "csrc")


def test_wide_and_large_images_are_refused(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "limits")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-pthread",
                        "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        os.path.join(CSRC, "plan_builder.cpp"),
                        os.path.join(CSRC, "stream_builder.cpp"),
                        os.path.join(ROOT, "tests", "sanitize", "stream_limits_harness.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
