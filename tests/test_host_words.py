"""Host-side check of the page-locked result words of the waiting calls
(csrc/host_words.h), compiled with g++ against a stand-in for the HIP runtime:
disjoint bounded slots, several threads, a page lost to a device reset, an
address taken by another allocation, other devices, capturing streams."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2003_07968_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "host_words_check.cpp")
ROCM_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_host_words_against_a_runtime_stand_in(tmp_path):
    exe = str(tmp_path / "host_words_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-D__HIP_PLATFORM_AMD__",
                    "-I", CSRC, "-I", ROCM_INCLUDE, SRC, "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr
