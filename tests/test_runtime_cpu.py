"""Host parts of libsal's runtime (scratch sizes, the kept device blocks on a
stand-in for the card, the tuner's keys, the forms of a batch), built with g++
under AddressSanitizer and UndefinedBehaviorSanitizer.  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2203_10000_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("rt") / "runtime_driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "sanitize", "runtime_driver.cpp"),
                        os.path.join(CSRC, "devmem.cpp"), os.path.join(CSRC, "tune_cache.cpp"),
                        "-lpthread", "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


def _run(driver, *check):
    r = subprocess.run([driver, *check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr[-4000:]


def test_scratch_for_n_points_holds_every_smaller_call(driver):
    _run(driver, "scratch")


def test_kept_blocks_are_a_reserve_of_every_allocation(driver):
    _run(driver, "reserve")


@pytest.mark.parametrize("check", ["streams", "threads"])
def test_kept_blocks_do_not_make_streams_or_threads_wait(driver, check):
    _run(driver, check)


def test_tuned_sizes_are_kept_by_form_and_surfaces(driver, tmp_path):
    _run(driver, "tuner", str(tmp_path / "tune.txt"))


def test_forms_of_a_batchs_instances(driver):
    _run(driver, "batch")
