"""161 to 192 columns of B on the chunk kernels, three tiles of 64 columns in one launch, against the CPU oracle
(needs the GPU)."""
import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

from test_gpu_parity import gpu_product, torch_gpu  # noqa: F401  (fixture)
from test_gpu_tiles import integer_matrix
from test_zz_no_alloc import _both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [160, 161, 163, 177, 188, 191, 192, 193])
@pytest.mark.parametrize("kw", [dict(ufi=1), dict(ufi=2), dict(ufi=4), dict(ufi=8), dict(ufi=8, sort_rows=1), dict(ufi=4, depth=1),
                                dict(ufi=4, cross=1, group_nnz=64), dict(ufi=2, force_wide=True), dict(kslices=2, ufi=4)],
                         ids=lambda kw: "-".join("%s%d" % i for i in kw.items()))
def test_bit_exact_on_integer_data(torch_gpu, oracle, kw, N):  # noqa: F811
    """Both sides of the rule's ends, last lanes with one to four columns, panels in several workgroups, and the
    plans that keep other tiles (64-bit addresses, column ranges)."""
    csr = integer_matrix(75, 1100, 0.3, 5 + N)
    B = np.random.default_rng(N).integers(-16, 17, (csr.K, N)).astype(np.float32)
    C, plan = gpu_product(torch_gpu, csr, B, guard_rows=2, **kw)
    assert plan.describe()["ufi"] == kw["ufi"] and (plan.describe()["n_cross"] > 0) == ("cross" in kw)
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B)
    assert np.abs(C_ref).max() < 2 ** 24
    assert np.array_equal(C.astype(np.float64), C_ref)
    if "kslices" not in kw:   # (refused there)
        for C2 in _both(torch_gpu, plan, B):
            assert np.array_equal(C, C2)


@pytest.mark.parametrize("M,K,N", [(700, 900, 161), (1500, 1500, 188), (1500, 1500, 192)])
def test_single_rows_on_both_sides_of_the_rule(torch_gpu, oracle, M, K, N):  # noqa: F811
    """Fewer and more than 2^19 entries, rows of B in and out of step with cache lines; also a last row of B
    at the very end of its allocation."""
    csr = gen.uniform_positions(M, K, 0.7, M + N)
    B = gen.dense_activations(K, N, 3)
    C, _ = gpu_product(torch_gpu, csr, B, guard_rows=2, ufi=1)
    C_ref, S = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B, parallel=True)
    err, bad_zero = oracle.parity_error(C, C_ref, S)
    assert bad_zero == 0 and err <= 1e-5
