"""Device memory kept between calls (workspace.cpp), on the CPU: the allocator
calls of the HIP runtime are replaced by a device of a few MiB, so that running
out of memory is an ordinary case (tests/workspace_check.cpp holds the checks)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1204_3425_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++") or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    out = str(tmp_path_factory.mktemp("workspace") / "check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-I", CSRC, "-I",
                           os.path.join(ROCM, "include"), os.path.join(HERE, "workspace_check.cpp"),
                           os.path.join(CSRC, "workspace.cpp"), "-o", out, "-pthread"])
    return out


@pytest.mark.parametrize("check", ["others_make_room", "lifetimes", "threads", "basis", "bound", "turns"])
def test_workspace(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
