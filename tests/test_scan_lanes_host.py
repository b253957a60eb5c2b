"""The scans whose waves share each column's second-best key, dense columns and wide
blocks with their conformations split, on emulated lanes: tests/host/emulator
runs the lanes of a workgroup on the CPU in a random order between the
operations that a wave does together, so that lanes of one column read the key at
different times.  Every phenotype, energy and gap is a whole number and has to
equal the count over all conformations.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CLANG = "/opt/rocm/llvm/bin/clang++"      # the kernels' vector types need clang


def test_scans_whatever_the_order_of_lanes(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++")
    csrc = os.path.join(ROOT, "paper_2008_05612_amd", "csrc")
    exe = str(tmp_path / "scan_driver")
    subprocess.check_call([CLANG, "-std=c++17", "-O2", "-Wno-psabi",
                           "-I" + os.path.join(HOST, "emulator"),
                           "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
                           os.path.join(HOST, "scan_driver.cpp"),
                           os.path.join(HOST, "emulator", "emulator.cpp"),
                           os.path.join(csrc, "structures.cpp"), "-o", exe, "-lpthread"])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    assert out.stdout == "dense 0 0 tables 0 0 wide 0 0 tables 0\n"
