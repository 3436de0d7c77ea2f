"""Bounds and coverage of the page write's items, on the CPU.

Pages that are counted by tokens find their row by a search over cu_new. The check
compiles the library's own item arithmetic for the host and runs it over lengths in order,
slices of a longer cu_new (cu_new[0] > 0) and cu_new in no order at all.
"""
import os
import subprocess

from paper_2603_18815_amd.build import CSRC, HIPCC, INCLUDE

HERE = os.path.dirname(os.path.abspath(__file__))


def test_items_stay_in_the_block_table(tmp_path):
    exe = tmp_path / "page_items_check"
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", INCLUDE,
                        "-I", CSRC, os.path.join(HERE, "page_items_check.cpp"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
