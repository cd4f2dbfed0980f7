"""The host code around allocations, read-outs and launch order (CPU only).

tests/sanitize/pool_driver.cpp is a HIP runtime made of host memory and the
library's host sources compiled with it under AddressSanitizer and
UndefinedBehaviorSanitizer: every allocation that an admission, a run of more
slots than before, a channel's creation or its tuning makes fails in turn, and
what was there before must still be stepped and read out through valid memory; a
read-out's arrays are written by the kernel only where that holds up no steps;
and every tile of a step is taken once, in the stated order."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1803_01756_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("pool") / "pool_driver")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-w",
                        "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                        "-I", CSRC, "-o", exe, os.path.join(HERE, "sanitize", "pool_driver.cpp"),
                        os.path.join(CSRC, "lbm_runtime.cpp"), os.path.join(CSRC, "lbm_pool.cpp")],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return exe


def _run(driver, what):
    r = subprocess.run([driver, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                       timeout=300)
    print(r.stdout)
    assert r.returncode == 0 and "0 failed expectations" in r.stdout, r.stdout


@pytest.mark.parametrize("what", ["first", "admission", "run"])
def test_failed_allocation_leaves_the_pool_usable(driver, what):
    _run(driver, what)


def test_creation_without_memory(driver):
    _run(driver, "create")


def test_failed_allocation_is_not_reported_by_another_channel(driver):
    _run(driver, "channel")


def test_admission_frees_nothing_while_the_batch_may_run(driver):
    _run(driver, "growth")


def test_readout_beside_a_running_batch_is_copied(driver):
    _run(driver, "readout")


def test_adjoining_pinned_arrays_are_copied_at_once(driver):
    _run(driver, "merge")


def test_every_tile_is_taken_once_in_the_stated_order(driver):
    _run(driver, "order")
