"""The choice of index entries and the memory set aside for them, checked on the
CPU over hash ranges, loads and capacities.  Compiles
tests/native/index_fmt_check.hip with hipcc (host code only runs)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_entries_fit_the_memory_of_the_capacities(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "index_fmt_check")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1907_02900_amd", "csrc"),
                           os.path.join(ROOT, "tests", "native", "index_fmt_check.hip"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout
