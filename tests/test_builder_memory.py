"""Host memory that runs out while the stream encoding is built (CPU only)."""
import os
import shutil
import subprocess

import pytest

from tests.helpers import ROOT

CSRC = os.path.join(ROOT, "paper_1412_6367_amd", "csrc")


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("memory") / "harness")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-pthread",
                        os.path.join(CSRC, "plan_builder.cpp"),
                        os.path.join(CSRC, "stream_builder.cpp"),
                        os.path.join(ROOT, "tests", "sanitize", "builder_memory_harness.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("npt,npt_azim", [(150, 0), (60, 36)])
def test_builder_out_of_memory(npt, npt_azim, harness):
    r = subprocess.run([harness, str(npt), str(npt_azim)], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.returncode, r.stdout + r.stderr)
