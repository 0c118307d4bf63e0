"""The C ABI's host code over a fake device (CPU only): what is left after a
set-up that runs out of memory half-way, and which kernels a pass takes."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from tests.helpers import ROOT

CSRC = os.path.join(ROOT, "paper_1412_6367_amd", "csrc")
SANITIZE = os.path.join(ROOT, "tests", "sanitize")
BUILD = "_ZN3azi12build_streamERKNS_10HostMatrixEiiillRNS_12StreamMatrixE"


@pytest.fixture(scope="module")
def over_fake_device(tmp_path_factory):
    """Links a harness with the C ABI's host code and the fake device."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    tmp = tmp_path_factory.mktemp("fake")

    def compile_one(src):
        obj = str(tmp / (os.path.basename(src) + ".o"))
        r = subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-w",
                            "-D__HIP_PLATFORM_AMD__", "-D__align__(x)=", "-DHIP_SYMBOL(x)=(&x)",
                            "-I/opt/rocm/include", "-fsanitize=address", "-x", "c++", "-c", src,
                            "-o", obj], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return obj

    common = [os.path.join(CSRC, "azint_api.hip"), os.path.join(CSRC, "plan_builder.cpp"),
              os.path.join(CSRC, "stream_builder.cpp"), os.path.join(SANITIZE, "fake_device.cpp")]
    with ThreadPoolExecutor(4) as pool:
        objects = list(pool.map(compile_one, common))

    def link(harness):
        exe = str(tmp / harness)
        r = subprocess.run(["g++", "-fsanitize=address", "-pthread", f"-Wl,--wrap={BUILD}", *objects,
                            compile_one(os.path.join(SANITIZE, harness + ".cpp")), "-o", exe],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return exe

    return link


@pytest.fixture(scope="module")
def harness(over_fake_device):
    return over_fake_device("corrections_harness")


@pytest.mark.parametrize("two_d,dtype,stage", [
    (1, 0, -1), (1, 1, -1),                     # maps
    (0, 0, -1), (0, 1, -1), (0, 0, 3), (0, 0, 4)])  # profiles: summed dark, fused, folded
def test_frames_after_a_failed_call_are_corrected(two_d, dtype, stage, harness):
    r = subprocess.run([harness, str(two_d), str(dtype), str(stage)], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr


@pytest.fixture(scope="module")
def encodings(over_fake_device):
    return over_fake_device("encodings_harness")


@pytest.mark.parametrize("kind", [0, 1, 2], ids=["map", "profile", "batch"])
def test_a_failed_retiling_leaves_a_whole_encoding(kind, encodings):
    r = subprocess.run([encodings, str(kind)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("ok"), (r.returncode, r.stdout + r.stderr)


@pytest.fixture(scope="module")
def routes(over_fake_device):
    return over_fake_device("routes_harness")


def kernels(routes, h, w, npt, npt_azim=0, dtype=0, n=0):
    r = subprocess.run([routes, *map(str, (h, w, npt, npt_azim, dtype, n))], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout.strip()


ROWS = "image forward, raw correct forward, backward backward"
MAP = "image stream, raw stream, backward backward"


@pytest.mark.parametrize("shape,passes", [
    ((330, 330, 100, 36), ROWS),             # encoding it would take longer than building it
    ((1413, 1415, 140, 12), ROWS),           # a row short of the line
    ((1414, 1415, 140, 12), MAP),
    ((1450, 1450, 450, 360), "image forward, raw stream, backward backward"),
    ((1450, 1450, 150, 720), ROWS),          # 1.6 entries a pixel, half a wedge a column
    ((1450, 1450, 1450, 720), ROWS),         # 2.5 entries per partial sum or item
], ids=str)
def test_map_passes(shape, passes, routes):
    assert kernels(routes, *shape) == passes


STREAM = "image stream, raw stream, backward stream_adjoint"
RUNS = "image band, raw band, backward backward"


@pytest.mark.parametrize("shape,passes", [
    ((1, 262144, 100), STREAM),              # 4096 tiles
    ((1, 262145, 100), RUNS),                # one more
    ((11, 262145, 100), RUNS),
    ((12, 262145, 100), STREAM),             # tiles of 12 rows
    ((300, 1, 40), STREAM),
    ((300, 300, 600), STREAM),               # 4.7 entries a pixel
    ((300, 300, 640), RUNS),                 # 4.9
    ((1740, 1740, 4350), STREAM),            # 5.6, three million pixels
    ((1740, 1740, 4900), RUNS),              # 6.2
], ids=str)
def test_passes_of_few_rows_and_of_fine_bins(shape, passes, routes):
    assert kernels(routes, *shape) == passes


@pytest.mark.parametrize("n,shape,passes", [
    (64, (1, 4096, 60), "image stream, backward stream_adjoint"),  # 4096 tiles together
    (65, (1, 4096, 60), "image band, backward backward"),
    (1000, (3, 130, 20), "image stream, backward stream_adjoint"),  # not wide
    (1000, (12, 1025, 20), "image stream, backward stream_adjoint"),
    (40, (60, 60, 120), "image stream, backward stream_adjoint"),
    (40, (60, 60, 130), "image band, backward backward"),
], ids=str)
def test_batch_passes_of_few_rows_and_of_fine_bins(n, shape, passes, routes):
    assert kernels(routes, *shape, n=n) == passes


@pytest.mark.parametrize("last,said", [
    ((20, 30, 0), "image stream, 50 encoded"),
    ((1, 3, 0), "image band, 0 encoded"),
    ((20, 30, 6), "image band, 0 encoded"),
], ids=str)
def test_a_refused_instance_is_seen_before_the_others_are_encoded(last, said, over_fake_device):
    r = subprocess.run([over_fake_device("mixed_batch_harness"), "50", *map(str, last)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == said, r.stdout + r.stderr
