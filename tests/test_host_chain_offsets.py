"""Offsets of the chained products' lists (kernels.h) in blocks larger than 32
bits of bytes: builds tests/cpp/chain_offsets_check.cpp and runs it on the
CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1703_04789_amd", "csrc")


def test_lane_offsets_reach_the_end_of_large_blocks(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    exe = str(tmp_path / "chain_offsets_check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + CSRC, "-I" + os.path.join(rocm, "include"),
                    os.path.join(ROOT, "tests", "cpp", "chain_offsets_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr
