"""Host logic of the library on a HIP runtime that books allocations and launches and computes nothing
(tests/host/fake_hip.cpp): launch limits, launch counts and memory held, without a GPU."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
LIB = os.path.join(ROOT, "paper_2609_00049_amd", "librealq.so")

pytestmark = [pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++"),
              pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")]


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Werror",
                    os.path.join(HOST, "fake_hip.cpp"), "-o", str(so)], check=True, capture_output=True, text=True)
    return str(so)


@pytest.mark.parametrize("check", ["whole_lines", "many_tokens", "short_chunks", "slice_memory", "little_room", "under_capture"])
def test_on_a_runtime_that_only_books(fake, check):
    res = subprocess.run([sys.executable, os.path.join(HOST, "host_logic.py"), fake, LIB, check], capture_output=True,
                         text=True, timeout=120)
    assert res.returncode == 0 and "passed" in res.stdout, res.stdout + res.stderr
