"""The allocation-free entry point allocates nothing in the set-up of a grid, on
the CPU: the library's host code with a counting heap (tests/hoststub)."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_set_up_allocates_nothing(tmp_path):
    if not os.path.exists(HIPCC) or shutil.which("g++") is None:
        pytest.skip("no hipcc or g++")
    obj, exe = str(tmp_path / "alloc.o"), str(tmp_path / "alloc")
    subprocess.run([HIPCC, "-O0", "-std=c++17", "--offload-host-only", "--offload-arch=gfx950", "-x", "hip", "-c",
                    os.path.join(ROOT, "tests", "hoststub", "alloc_driver.cpp"), "-o", obj], check=True)
    subprocess.run(["g++", "-no-pie", obj, "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
