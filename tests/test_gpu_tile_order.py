"""Order in which the workgroups of several column tiles start: every block of every tile exactly once, against the
CPU oracle (needs the GPU)."""
import numpy as np
import pytest

from test_gpu_parity import gpu_product, torch_gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


class Matrix:
    """Rows of the given lengths, small whole numbers."""

    def __init__(self, lengths, K, seed):
        rng = np.random.default_rng(seed)
        self.M, self.K = len(lengths), K
        self.row_ptr = np.concatenate(([0], np.cumsum(lengths))).astype(np.int32)
        self.col_idx = np.concatenate([np.sort(rng.choice(K, n, replace=False)) for n in lengths]).astype(np.int32)
        self.vals = rng.integers(1, 9, len(self.col_idx)).astype(np.float32)


MATRICES = {"even-few": lambda: Matrix([40] * 300, 500, 1),                            # fewer blocks than one per unit and tile
            "even-many": lambda: Matrix([64] * 9000, 400, 2),
            "uneven-few": lambda: Matrix([700] * 3 + [20] * 400, 700, 3),
            "uneven-many": lambda: Matrix([900] * 40 + [30] * 12000, 900, 4)}


@pytest.mark.parametrize("N", [129, 176, 200, 239, 240, 256, 384, 511, 1024, 1100])
@pytest.mark.parametrize("kw", [dict(ufi=1), dict(ufi=4), dict(ufi=8, cross=1, group_nnz=64), dict(n_hint=32), dict(n_hint=16)],
                         ids=lambda kw: "-".join("%s%d" % i for i in kw.items()))
@pytest.mark.parametrize("name", list(MATRICES))
def test_bit_exact_on_integer_data(torch_gpu, oracle, name, kw, N):  # noqa: F811
    """Two, three, four, eight and more tiles, whole and partial last ones, tiles of 128, 64, 32 and 16 columns."""
    csr = MATRICES[name]()
    B = np.random.default_rng(N).integers(-16, 17, (csr.K, N)).astype(np.float32)
    C, _ = gpu_product(torch_gpu, csr, B, guard_rows=1, tiles=-1, **kw)
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B, parallel=True)
    assert np.abs(C_ref).max() < 2 ** 24
    assert np.array_equal(C.astype(np.float64), C_ref)
