"""The library's host sources on stand-ins for the HIP runtime and the kernels (tests/host_sources_on_stand_ins.cpp):
what runs only where memory is short, and what the executor hands to the launcher."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2506_15174_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_sources") / "host_sources")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(rocm, "include"), os.path.join(HERE, "host_sources_on_stand_ins.cpp"),
                    os.path.join(CSRC, "spmm_api.cpp"), os.path.join(CSRC, "spmm_plan.cpp"), "-pthread", "-o", exe], check=True)
    return exe


def passes(program, what):
    res = subprocess.run([program, what], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.endswith("ok\n"), res.stdout + res.stderr


def test_failed_allocations_are_a_status(program):
    """A status, no exception, nothing left behind."""
    passes(program, "failures")


def test_which_path_is_chosen(program):
    passes(program, "choices")


def test_blocks_are_dealt_or_compute_units_held_to_two_workgroups(program):
    passes(program, "launches")


def test_every_block_of_every_column_tile_once(program):
    passes(program, "places")


def test_rows_out_of_order_are_sorted_by_several_threads(program):
    passes(program, "threads")
