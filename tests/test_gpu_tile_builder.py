"""Building tiles with the bitmaps of a panel in LDS and, for more than 1024 steps, in global memory (needs the GPU)."""
import numpy as np
import pytest

import paper_2506_15174_amd as spmm

from test_gpu_parity import torch_gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [8, 16, 32])
@pytest.mark.parametrize("steps", [1, 2, 63, 64, 65, 1023, 1024, 1025])
def test_panels_of_up_to_as_many_steps_as_threads(torch_gpu, tiles, steps):  # noqa: F811
    """Rows cut short, an empty row and a dense one; a column twice and one outside are found in either memory."""
    torch = torch_gpu
    K = steps * 1024 // tiles - 3
    M = tiles + tiles // 2
    rng = np.random.default_rng(steps)
    lens = rng.integers(0, min(K, 700), M)
    lens[1], lens[tiles] = 0, min(K, 20000)
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col_idx = np.concatenate([rng.choice(K, n, replace=False) for n in lens]).astype(np.int32)
    vals = rng.integers(-8, 9, len(col_idx)).astype(np.float32)
    plan = spmm.plan_create(M, K, row_ptr, col_idx, vals, tiles=tiles)
    assert plan.describe()["tile_rows"] == tiles
    B = torch.randint(-8, 9, (K, 4), device="cuda", dtype=torch.int8).to(torch.float32)
    rows = torch.from_numpy(np.repeat(np.arange(M), lens)).cuda()
    terms = torch.from_numpy(vals).cuda().double()[:, None] * B[torch.from_numpy(col_idx).cuda().long()].double()
    want = torch.zeros((M, 4), device="cuda", dtype=torch.float64).index_add_(0, rows, terms)
    assert torch.equal(plan.execute(B).double(), want)
    at = int(row_ptr[tiles]) + 5 if lens[tiles] > 6 else 0
    twice = col_idx.copy()
    twice[at + 1] = twice[at]
    assert spmm.plan_create(M, K, row_ptr, twice, vals, tiles=tiles).describe()["tile_rows"] == 0
    for outside in (-1, K):
        bad = col_idx.copy()
        bad[at] = outside
        with pytest.raises(spmm.SpmmError) as err:
            spmm.plan_create(M, K, row_ptr, bad, vals, tiles=tiles)
        assert err.value.status == spmm.SPMM_ERR_INVALID_CSR
