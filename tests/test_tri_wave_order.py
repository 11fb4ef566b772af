"""The triangle limiter's decisions do not depend on the order in which a block's waves run.

The kernel source is compiled as host code and run by a small block emulator
(tests/block_emulator): every wave runs up to the next block barrier before the next
wave of the chosen order starts, for every order.  A flag in LDS that one wave clears
and another sets without a barrier between the two shows as a decision that is lost
under some order."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EMU = os.path.join(ROOT, "tests", "block_emulator")
CSRC = os.path.join(ROOT, "paper_2112_05946_amd", "csrc")


def test_limiter_decision_under_every_wave_order(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "tri_limiter")
    cmd = [cxx, "-std=c++17", "-O1", "-w", "-I" + EMU, "-I" + CSRC, "-I" + os.path.join(ROOT, "include"),
           "-include", os.path.join(EMU, "hip", "hip_runtime.h"), "-x", "c++", os.path.join(EMU, "tri_limiter.cpp"),
           os.path.join(CSRC, "tables.cpp"), os.path.join(CSRC, "tables_tri.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
