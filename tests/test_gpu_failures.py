"""Calls that fail in the middle (memory runs out, a kernel never runs): what
they return and what they leave behind.  Each case runs in a process of its
own, whose HIP calls go through hip_shim.cpp."""
import os
import subprocess
import sys

import pytest

from gpu_failing import OPTIONS

pytestmark = pytest.mark.gpu
TESTS = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("shim") / "hip_shim.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(TESTS, "hip_shim.cpp"), "-ldl"], check=True)
    return so


def _run(shim, case):
    print(f"case: {case}", flush=True)
    r = subprocess.run([sys.executable, os.path.join(TESTS, "gpu_failing.py"), shim, case],
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    print(r.stdout, flush=True)


@pytest.mark.parametrize("case", sorted(OPTIONS))
def test_batch_out_of_memory(shim, case):
    _run(shim, f"oom:{case}")


def test_server_goes_on_after_failed_batches(shim):
    _run(shim, "server")
