"""The serving loop's host code over a stand-in for the HIP runtime and the
plans (``serve_stub.cpp``): a step that fails ends its own request, releases
its plan and leaves the server running; partial sums that a dense plan could
do without keep no request from running beside others."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1206_0115_amd", "csrc")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not installed")
    exe = str(tmp_path_factory.mktemp("serve") / "serve_stub")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + CSRC, "-I" + os.path.join(ROOT, "include"),
                    os.path.join(HERE, "serve_stub.cpp"), os.path.join(CSRC, "serve.cpp"),
                    "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("what", ["upload", "wait", "precision"])
def test_failed_step_ends_its_request(stub, what):
    r = subprocess.run([stub, what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_partial_sums_keep_no_request_waiting(stub):
    r = subprocess.run([stub, "beside"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
