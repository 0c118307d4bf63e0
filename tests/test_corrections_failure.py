"""Corrections whose set-up runs out of memory half-way (CPU only, the C ABI
over a fake device): frames integrated afterwards are still corrected."""
import os
import shutil
import subprocess

import pytest

from tests.helpers import ROOT

CSRC = os.path.join(ROOT, "paper_1412_6367_amd", "csrc")
SANITIZE = os.path.join(ROOT, "tests", "sanitize")


def compile_over_fake_device(exe, *sources):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-pthread", "-w",
                        "-D__HIP_PLATFORM_AMD__", "-D__align__(x)=", "-DHIP_SYMBOL(x)=(&x)",
                        "-I/opt/rocm/include", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-x", "c++",
                        os.path.join(CSRC, "azint_api.hip"),
                        os.path.join(CSRC, "plan_builder.cpp"),
                        os.path.join(CSRC, "stream_builder.cpp"),
                        os.path.join(SANITIZE, "fake_device.cpp"),
                        *(os.path.join(SANITIZE, s) for s in sources), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    return compile_over_fake_device(str(tmp_path_factory.mktemp("corr") / "harness"),
                                    "corrections_harness.cpp")


@pytest.mark.parametrize("two_d,dtype,stage", [
    (1, 0, -1), (1, 1, -1),                     # maps
    (0, 0, -1), (0, 1, -1), (0, 0, 3), (0, 0, 4)])  # profiles: summed dark, fused, folded
def test_frames_after_a_failed_call_are_corrected(two_d, dtype, stage, harness):
    r = subprocess.run([harness, str(two_d), str(dtype), str(stage)], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
