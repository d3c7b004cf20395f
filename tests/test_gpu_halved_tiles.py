"""Chunk plans whose fullest compute unit is spared enough by it: 97 to 128 columns run as two tiles of 64, 41 to 64
as two of 32, other widths in one.  Small integers: every order of the sums is exact."""
import ctypes

import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

pytestmark = pytest.mark.gpu


# A few rows hold most entries (they are cut into pieces); rows of two lengths; panels of two rows; even rows of 75 blocks, for which half of
# the units would be idle, and of 256; rows for chunks of more columns; a row alone; and a pipeline depth asked for.  `halved`: a 1 for 41 to 64 columns in two
# tiles, a 2 for 97 to 119, a 4 for 120 to 128.
@pytest.mark.parametrize("M,K,lengths,kw,halved", [
    (300, 4096, (2000, 40), {}, 7), (500, 900, (700, 20), dict(n_hint=128), 6), (256, 3000, (900, 300), dict(ufi=2), 6), (600, 800, (30, 30), dict(n_hint=100), 6),
    (1024, 2048, (200, 200), dict(n_hint=128), 0), (200, 9000, (8000, 20), dict(n_hint=64), 7), (500, 900, (700, 20), dict(n_hint=32), 0), (1, 5000, (4000, 0), {}, 7),
    (300, 4096, (2000, 40), dict(depth=1), 7)])
def test_whole_numbers_are_exact(M, K, lengths, kw, halved):
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(M)
    W = np.zeros((M, K), dtype=np.float32)
    for i in range(M):
        n = lengths[0] if i % 16 == 0 else lengths[1]
        W[i, rng.choice(K, n, replace=False)] = rng.integers(1, 5, n)
    csr = gen.csr_from_dense(W)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=-1, strips=-1, **kw)
    assert plan.describe()["tile_rows"] == 0 and plan.describe()["strip_units"] == 0
    f, cols = spmm.load().spmm_chunk_tiles, ctypes.c_int32(0)
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p]
    for N, tile, bit in ((40, 64, 0), (41, 64, 1), (64, 64, 1), (65, 128, 0), (96, 128, 0), (97, 128, 2), (119, 128, 2), (120, 128, 4), (128, 128, 4)):
        if plan.describe()["ufk"] != 8 or (N > 64 and 8192 < K <= 16384):  # other tiles anyway
            continue
        two = 2 if halved & bit else 1
        assert f(plan.handle, N, ctypes.byref(cols)) == two and cols.value * two == tile, N
    for N in (33, 40, 41, 48, 63, 64, 65, 96, 97, 100, 119, 120, 127, 128, 129, 200, 256):
        B = rng.integers(-4, 5, (K, N)).astype(np.float32)
        full = torch.full((M + 2, N), float("nan"), device="cuda")
        for _ in range(2):
            plan.execute(torch.from_numpy(B).cuda(), full[1:M + 1])
            C = full.cpu().numpy()
            assert np.array_equal(C[1:M + 1], W @ B) and np.isnan(C[[0, M + 1]]).all(), N  # sums below 2^24
