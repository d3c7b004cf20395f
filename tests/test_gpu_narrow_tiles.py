"""Matrix-core path on panels of 8 rows (narrow B) against the CPU oracle, through the C ABI (needs the GPU)."""
import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

from test_gpu_parity import check, gpu_product, torch_gpu  # noqa: F401  (fixture)
from test_gpu_tiles import integer_matrix

pytestmark = pytest.mark.gpu


def bit_exact(torch_gpu, oracle, M, K, density, N):  # noqa: F811
    csr = integer_matrix(M, K, density, M + K)
    B = np.random.default_rng(N).integers(-16, 17, (K, N)).astype(np.float32)
    C, plan = gpu_product(torch_gpu, csr, B, guard_rows=2, tiles=8)
    assert plan.describe()["tile_rows"] == 8
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B)
    assert np.abs(C_ref).max() < 2 ** 24
    assert np.array_equal(C.astype(np.float64), C_ref)


@pytest.mark.parametrize("N", [1, 3, 4, 5, 16, 17, 70])
@pytest.mark.parametrize("density", [0.05, 0.3, 0.8])
@pytest.mark.parametrize("M,K", [(3, 1), (9, 129), (70, 1024), (130, 4225), (5, 70001)])
def test_panels_steps_and_runs_of_steps(torch_gpu, oracle, M, K, density, N):  # noqa: F811
    """Sizes no panel or step divides, fewer steps than waves, more than one run of 64 steps per wave;
    one, two and four loads per block; fewer columns than a tile and more."""
    bit_exact(torch_gpu, oracle, M, K, density, N)


@pytest.mark.parametrize("N", [4, 7, 8, 13, 16])
@pytest.mark.parametrize("M,K,density", [(1040, 4200, 0.1), (2056, 4200, 0.1), (4104, 300, 0.2), (4104, 4200, 0.05), (8200, 140, 0.6)])
def test_every_width_and_number_of_waves(torch_gpu, oracle, M, K, density, N):  # noqa: F811
    """Panels enough that all of a tile's widths and both workgroup sizes are taken."""
    bit_exact(torch_gpu, oracle, M, K, density, N)


def test_chosen_for_narrow_b(torch_gpu, oracle):  # noqa: F811
    csr = gen.uniform_positions(2048, 4096, 0.8, 1)
    for N in (4, 16):
        B = gen.dense_activations(4096, N, 3)
        C, plan = gpu_product(torch_gpu, csr, B, n_hint=N)
        assert plan.describe()["tile_rows"] == 8
        check(oracle, csr, B, C, parallel=True)
        assert gpu_product(torch_gpu, csr, B, n_hint=N, tiles=-1)[1].describe()["tile_rows"] == 0


def test_rows_of_b_too_long_for_32_bit_offsets(torch_gpu, oracle):  # noqa: F811
    """A step's rows of B span more than 4 GiB: 64-bit addresses.  Checked on columns at both ends."""
    torch = torch_gpu
    csr = integer_matrix(20, 33, 0.5, 9)
    N = (1 << 32) // (128 * 4) + 3
    B = torch.randint(-9, 10, (csr.K, N), device="cuda", dtype=torch.int8).to(torch.float32)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=8)
    C = plan.execute(B)
    cols = torch.cat([torch.arange(0, 200), torch.arange(N - 200, N)]).cuda()
    B_small, C_small = B[:, cols].contiguous().cpu().numpy(), C[:, cols].cpu().numpy()
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B_small)
    assert np.array_equal(C_small.astype(np.float64), C_ref)


def test_more_workgroups_than_one_launch_takes(torch_gpu, oracle):  # noqa: F811
    """C of 8 GiB on panels of 8 rows: 2^24 workgroups of 256 threads, one more launch than HIP takes at
    once.  All of C is compared, a run of columns at a time."""
    torch = torch_gpu
    M, N = 32768, 65536
    csr = integer_matrix(M, 16, 0.4, 31)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=8)
    assert plan.describe()["tile_rows"] == 8
    B = torch.randint(-9, 10, (csr.K, N), device="cuda").to(torch.float32)
    C = torch.full((M, N), float("nan"), device="cuda")
    plan.execute(B, C)
    A = np.zeros((M, csr.K), np.float32)
    A[np.repeat(np.arange(M), np.diff(csr.row_ptr)), csr.col_idx] = csr.vals
    A = torch.from_numpy(A).cuda()
    for j in range(0, N, 8192):   # small integers: every order of the sums is exact
        assert torch.equal(C[:, j:j + 8192], A @ B[:, j:j + 8192].contiguous()), j
    cols = np.r_[0:8, N - 8:N]
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B[:, cols].contiguous().cpu().numpy())
    assert np.array_equal(C[:, cols].cpu().numpy().astype(np.float64), C_ref)


def test_as_many_columns_as_the_interface_counts(torch_gpu):  # noqa: F811
    """N = 2^31 - 1: the number of column tiles is rounded up beyond 31 bits.  One row of A, so that
    C is a sum of scaled rows of B; all of it is compared, a run of columns at a time."""
    torch = torch_gpu
    N = 2 ** 31 - 1
    plan = spmm.plan_create(1, 2, np.array([0, 2]), np.array([0, 1]), np.array([3.0, -2.0]), tiles=8)
    assert plan.describe()["tile_rows"] == 8
    B = torch.empty((2, N), device="cuda")
    for j in range(0, N, 1 << 28):
        B[:, j:j + (1 << 28)] = torch.randint(-9, 10, B[:, j:j + (1 << 28)].shape, device="cuda", dtype=torch.int8)
    C = plan.execute(B)
    for j in range(0, N, 1 << 28):
        assert torch.equal(C[0, j:j + (1 << 28)], 3 * B[0, j:j + (1 << 28)] - 2 * B[1, j:j + (1 << 28)]), j
