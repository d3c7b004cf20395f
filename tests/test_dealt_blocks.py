"""Chunk plans whose blocks are dealt to the compute units: the order (on stand-ins for the device) and the products."""
import os
import subprocess

import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2506_15174_amd", "csrc")


def test_every_block_once_and_loads_more_even(tmp_path):
    exe = str(tmp_path / "dealt_blocks")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-I", HERE,
                    "-I", os.path.join(rocm, "include"), os.path.join(HERE, "dealt_blocks_on_stand_ins.cpp"),
                    os.path.join(CSRC, "spmm_api.cpp"), os.path.join(CSRC, "spmm_plan.cpp"), "-pthread", "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.endswith("ok\n"), res.stdout + res.stderr


# 256 blocks and a few, 512 and a few, up to four to a unit; two, four and eight slices, chunks of 16, panels of one and two
# rows; widths that leave lanes idle, and two column tiles, which keep the plan's own order.  Small integers: every order of the
# sums is exact.
@pytest.mark.gpu
@pytest.mark.parametrize("M,K,density,hint,widths", [
    (1024, 2048, 0.10, 64, (64, 33, 128, 200)),
    (1024, 4096, 0.10, 64, (64, 1, 32)),
    (2048, 4096, 0.10, 32, (32, 17)),
    (700, 5000, 0.10, 100, (100, 128)),
    (5000, 2000, 0.03, 128, (128, 64)),
    (896, 1024, 0.08, 0, (105, 160)),
])
def test_products(M, K, density, hint, widths, oracle):
    import torch
    csr = gen.lognormal_rows(M, K, 1.0 - density, 5)
    vals = np.random.default_rng(6).integers(-8, 9, csr.vals.size).astype(np.float32)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, vals, n_hint=hint, tiles=-1, strips=-1)
    info = plan.describe()
    assert 256 < info["n_blocks"] <= 1024
    for N in widths:
        B = np.random.default_rng(N).integers(-16, 17, (K, N)).astype(np.float32)
        got = plan.execute(torch.from_numpy(B).cuda(), torch.full((M, N), float("nan"), device="cuda"))
        want, _ = oracle.spmm(csr.row_ptr, csr.col_idx, vals, B)
        assert np.array_equal(got.cpu().numpy(), want.astype(np.float32))
