"""The library's host code (csrc/pd_api.hip and the launchers) run on the CPU, over a stand-in for the HIP runtime: what a
call leaves behind when one of its launches or allocations fails, and which launches the largest calls make."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_2603_04716_amd")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launches") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wno-missing-field-initializers", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host_launches_driver.cpp"),
                    os.path.join(LIB_DIR, "libpd_mi355x.so"), "-rdynamic", f"-Wl,-rpath,{LIB_DIR}",
                    "-Wl,--unresolved-symbols=ignore-in-shared-libs", "-o", exe], check=True)
    return exe


def run(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


def test_a_failed_call_leaves_the_cache_lengths_alone(driver):
    run(driver, "failures")


def test_rows_near_the_size_limit_of_a_launch(driver):
    run(driver, "limits")
