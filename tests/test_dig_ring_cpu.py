"""Addresses that the digit product's record copies ask for, on the CPU: tests/dig_ring_sweep.cpp walks the ring with the
very functions that the kernel and the allocation use (csrc/bbmm_plan.h)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_record_copies_stay_inside_their_buffer(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path / "dig_ring_sweep"
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1809_11165_amd", "csrc"),
                    os.path.join(ROOT, "tests", "dig_ring_sweep.cpp"), "-o", str(exe)], check=True)
    proc = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert proc.returncode == 0, proc.stderr[-2000:]
    assert proc.stdout.startswith("OK ")
