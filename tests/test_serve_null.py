"""The serving loop's HIP backend, compiled for the host, on a null device
(CPU only): an error of the runtime ends the requests that it belongs to."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1911_13225_amd", "csrc")
ROCM = "/opt/rocm/include"


@pytest.fixture(scope="module")
def binary(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(os.path.join(ROCM, "hip")):
        pytest.skip("needs g++ and the HIP headers")
    out = str(tmp_path_factory.mktemp("serve") / "serve_null")
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", ROCM, "-I", CSRC,
           "-I", os.path.join(ROOT, "include"), "-x", "c++", os.path.join(CSRC, "serve.hip"),
           os.path.join(ROOT, "tests", "sched", "serve_null.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


@pytest.mark.parametrize("scenario", ["copy", "launch"])
def test_an_error_ends_the_requests_it_belongs_to(binary, scenario):
    """copy: a failing copy of one request's code leaves a running request, and
    one submitted later, to end DIST_OK.  launch: a failing launch of the tick
    ends the running request with DIST_EHIP, and a later one ends DIST_OK."""
    r = subprocess.run([binary, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-4000:])
    assert f"ok {scenario}" in r.stdout
