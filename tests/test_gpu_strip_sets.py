"""Strips in two sets, each fetched by half of the XCDs: every strip of every group of rows is computed once, at sets of equal
and of different sizes, in one band and in several, in one round of workgroups and in more."""
import ctypes

import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

pytestmark = pytest.mark.gpu


# 16 strips are the fewest in sets; 20 and 36 come in sets of 12 and 8, 20 and 16; 120 and 136 columns in one.
@pytest.mark.parametrize("N", [120, 128, 136, 160, 192, 256, 288, 2080])
@pytest.mark.parametrize("M,K,density", [(3, 2500, 0.3), (257, 3000, 0.02), (1500, 2048, 0.03), (700, 6000, 0.02)])
def test_whole_numbers_are_exact(M, K, density, N):
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(M + N)
    W = np.where(rng.random((M, K)) < density, rng.integers(1, 5, (M, K)), 0).astype(np.float32)
    csr = gen.csr_from_dense(W)
    B = rng.integers(-4, 5, (K, N)).astype(np.float32)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, n_hint=128, strips=1)
    info = plan.describe()
    assert info["strip_units"] > 0
    f = spmm.load().spmm_strips_of_set
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int32]
    first = {128: 8, 160: 12, 192: 12, 256: 16, 288: 20, 2080: 132}.get(N, (N + 7) // 8)
    assert f(info["n_enum"] // 64, K, N) == first
    full = torch.full((M + 2, N), float("nan"), device="cuda")
    for _ in range(2):
        plan.execute(torch.from_numpy(B).cuda(), full[1:M + 1])
        C = full.cpu().numpy()
        assert np.array_equal(C[1:M + 1], W @ B) and np.isnan(C[[0, M + 1]]).all()  # sums of whole numbers below 2^24
