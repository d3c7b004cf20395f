"""Column tiles of panels of 16 rows in two sets, each fetched by half of the XCDs: every tile of every panel is computed once, at
sets of equal and of different sizes, for tiles of 16, 32 and 64 columns, and where one set is left."""
import ctypes

import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

pytestmark = pytest.mark.gpu


# Two sets: rows of whole lines (multiples of 32 columns), more than a line of tiles, blocks of less than 1.5 times B's bytes (of the
# fourth matrix at the widest only).
@pytest.mark.parametrize("N", [32, 64, 96, 128, 132, 160, 224, 256, 1056])
@pytest.mark.parametrize("M,K,density", [(1, 640, 0.3), (17, 2050, 0.1), (300, 1500, 0.05), (2100, 300, 0.2), (40, 700, 0.9)])
def test_whole_numbers_are_exact(M, K, density, N):
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(M + N)
    W = np.where(rng.random((M, K)) < density, rng.integers(1, 5, (M, K)), 0).astype(np.float32)
    csr = gen.csr_from_dense(W)
    B = rng.integers(-4, 5, (K, N)).astype(np.float32)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, n_hint=N, tiles=16)
    info = plan.describe()
    assert info["tile_rows"] == 16
    f = spmm.load().spmm_tiles_of_set
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_int64]
    one = f(16, M, K, N, 1 << 62)  # all tiles
    first = f(16, M, K, N, info["stream_words"])
    assert (first < one) == (N % 32 == 0 and N > 32 and (M < 2100 or N > 256))
    full = torch.full((M + 2, N), float("nan"), device="cuda")
    for _ in range(2):
        plan.execute(torch.from_numpy(B).cuda(), full[1:M + 1])
        C = full.cpu().numpy()
        assert np.array_equal(C[1:M + 1], W @ B) and np.isnan(C[[0, M + 1]]).all()  # sums of whole numbers below 2^24
