"""The probe index entries of 32-bit keys, checked on the CPU: entries of
random buckets of every length, over hash ranges and loads that give every
field width and both entry sizes, against counting the bucket.  Compiles
tests/native/head_fmt_check.hip with hipcc (host code only runs)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_entries_answer_as_their_buckets(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "head_fmt_check")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1907_02900_amd", "csrc"),
                           os.path.join(ROOT, "tests", "native", "head_fmt_check.hip"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout
