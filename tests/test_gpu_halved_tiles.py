"""Chunk plans whose fullest compute unit has far more to do than the others: 97 to 128 columns run as two tiles of 64, 41 to 64
as two of 32, other widths in one.  Small integers: every order of the sums is exact."""
import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

pytestmark = pytest.mark.gpu


# A few rows hold most entries (they are cut into pieces); rows of two lengths; panels of two rows; even rows, which keep one tile; a
# row alone; and a pipeline depth asked for.
@pytest.mark.parametrize("M,K,lengths,kw", [(300, 4096, (2000, 40), {}), (500, 900, (700, 20), dict(n_hint=128)), (256, 3000, (900, 300), dict(ufi=2)),
                                            (600, 800, (30, 30), dict(n_hint=100)), (200, 9000, (8000, 20), dict(n_hint=64)), (1, 5000, (4000, 0), {}), (300, 4096, (2000, 40), dict(depth=1))])
def test_whole_numbers_are_exact(M, K, lengths, kw):
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
    for N in (33, 40, 41, 48, 63, 64, 65, 96, 97, 100, 119, 120, 127, 128, 129, 200, 256):
        B = rng.integers(-4, 5, (K, N)).astype(np.float32)
        full = torch.full((M + 2, N), float("nan"), device="cuda")
        for _ in range(2):
            plan.execute(torch.from_numpy(B).cuda(), full[1:M + 1])
            C = full.cpu().numpy()
            assert np.array_equal(C[1:M + 1], W @ B) and np.isnan(C[[0, M + 1]]).all(), N  # sums below 2^24
