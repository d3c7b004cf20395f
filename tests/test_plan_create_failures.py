"""Plan creation where host or device memory runs out: a status, no exception, nothing left behind.  A C++
program with stand-ins for the HIP runtime (tests/plan_create_failures.cpp) lets one allocation after the
other fail inside the library's own host sources."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2506_15174_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("failures") / "plan_create_failures")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(rocm, "include"), os.path.join(HERE, "plan_create_failures.cpp"),
                    os.path.join(CSRC, "spmm_api.cpp"), os.path.join(CSRC, "spmm_plan.cpp"), "-pthread", "-o", exe], check=True)
    return exe


def test_failed_allocations_are_a_status(program):
    res = subprocess.run([program], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.endswith("ok\n"), res.stdout + res.stderr
