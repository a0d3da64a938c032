"""The host side of the set and get calls (csrc/ppml_transfer.hpp), on the CPU:
built against a stand-in for the HIP runtime whose copies take effect only when
they are waited for (tests/hoststub), plain and under the thread and the address
sanitizer."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = os.path.join(ROOT, "tests", "hoststub")
BUILDS = {"plain": [], "thread": ["-fsanitize=thread"],
          "address": ["-fsanitize=address,undefined", "-fno-sanitize-recover=all"]}
CASES = ["sizes", "several_calls", "per_thread_stream", "record_fails", "environment", "devices", "held"]


@pytest.fixture(scope="module", params=list(BUILDS))
def driver(request, tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("transfer") / request.param)
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", *BUILDS[request.param], "-I", STUB,
                    os.path.join(STUB, "transfer_driver.cpp"), "-o", exe, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("case", CASES)
def test_transfer(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
