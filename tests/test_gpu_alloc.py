"""What the library allocates, and what it does where memory is short: cases in a process whose
HIP allocation calls are counted, and refused above a limit (tests/hip_shim.cpp)."""

import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))

CASES = ["shim", "noalloc", "exact_workspace", "exact_answer_without_distance_rows", "tries",
         "plan_tries"]


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("shim") / "hip_shim.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", "-o", so,
                           os.path.join(HERE, "hip_shim.cpp"), "-ldl"])
    return so


@pytest.mark.parametrize("case", CASES)
def test_allocation(shim, case):
    print(f"[alloc] {case}", flush=True)
    r = subprocess.run([sys.executable, "-u", os.path.join(HERE, "alloc_child.py"), shim, case], timeout=100,
                       capture_output=True, text=True)
    print(r.stdout, r.stderr[-3000:], flush=True)
    assert r.returncode == 0
