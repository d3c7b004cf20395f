"""The windows that a wave of the chunk kernel stages through LDS, at their edges: rows whose entries fill a whole number of
loads of 256 words, a little less or more, a whole window, and several windows one after the other."""
import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

pytestmark = pytest.mark.gpu


# A chunk of c columns of a single row takes 2 c words, its header one; headers are filled up to a multiple of eight.  So 15
# chunks of 8 take 256 words, 30 take 512, 45 (48 headers) 768, and 60 a window of 1024; of 16 and 64 columns 31 and 15 are a window at most.
@pytest.mark.parametrize("hint,columns", [(128, 8), (64, 8), (32, 16), (16, 32), (4, 64)])
def test_rows_at_the_edges_of_loads_and_windows(hint, columns):
    import torch
    assert torch.cuda.is_available()
    window = 1024 if columns < 32 else 2048

    def words(chunks):
        return (chunks + 7) // 8 * 8 + 2 * columns * chunks

    edges = [max(c for c in range(1, 200) if words(c) <= w) for w in range(256, window + 1, 256)]
    K = 4096
    lengths = sorted({min(K, max(1, m * e * columns + d)) for e in edges for d in (-1, 0, 1, columns) for m in (1, 2, 3)})
    rng = np.random.default_rng(hint)
    W = np.zeros((len(lengths), K), dtype=np.float32)
    for i, n in enumerate(lengths):
        W[i, rng.choice(K, n, replace=False)] = rng.integers(1, 5, n)
    csr = gen.csr_from_dense(W)
    B = rng.integers(-4, 5, (K, hint)).astype(np.float32)
    # a group takes whole rows of up to 1024 entries; longer ones are cut
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, n_hint=hint, ufi=1, group_nnz=1024, group_panels=16)
    info = plan.describe()
    assert info["ufk"] == columns and info["tile_rows"] == 0 and info["strip_units"] == 0
    for _ in range(2):
        C = plan.execute(torch.from_numpy(B).cuda()).cpu().numpy()
        assert np.array_equal(C, W @ B)  # sums of whole numbers below 2^24
