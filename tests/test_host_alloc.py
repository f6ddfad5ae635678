"""The library's memory handling on the CPU: its host code runs over a stand-in
for the HIP runtime (tests/native/fake_hip.h) that counts memory, fails
allocations on demand and runs no kernel."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1907_02900_amd")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    rocm = "/opt/rocm"
    if not os.path.exists(os.path.join(rocm, "include", "hip", "hip_runtime.h")):
        pytest.skip("no HIP headers")
    if not os.path.exists(os.path.join(PKG, "libhashgraph.so")):
        from paper_1907_02900_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("host") / "host_alloc_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-rdynamic",
                           "-w", "-I", os.path.join(rocm, "include"),
                           "-I", os.path.join(ROOT, "include"),
                           os.path.join(ROOT, "tests", "native", "host_alloc_check.cpp"),
                           os.path.join(PKG, "libhashgraph.so"), "-L", os.path.join(rocm, "lib"),
                           "-lamdhip64", "-Wl,-rpath," + PKG, "-Wl,-rpath," + rocm + "/lib",
                           "-o", exe])

    def run(what):
        r = subprocess.run([exe, what], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                           text=True, timeout=600)
        assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout[-2000:]
    return run


def test_rebuilds_within_the_capacity_allocate_nothing(check):
    check("rebuilds")


def test_a_failed_allocation_leaves_nothing_half_done(check):
    check("failures")


def test_the_pool_is_given_back(check):
    check("pool")


def test_intersections_take_no_builds_workspace(check):
    check("scatter")
