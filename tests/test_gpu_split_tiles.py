"""Panels of 32 rows x 128 and 64 columns on bf16 matrix instructions (values in three parts) against the CPU oracle,
through the C ABI (needs the GPU)."""
import ctypes

import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

from test_gpu_parity import gpu_product, torch_gpu  # noqa: F401  (fixture)
from test_gpu_tiles import integer_matrix

pytestmark = pytest.mark.gpu

WIDE = 128 * 128   # columns enough that one panel or two are multiplied in tiles of 128 columns


def column_groups(M, K, N):
    lib, nb = spmm.load(), ctypes.c_int(0)
    lib.spmm_tiles_time.restype = ctypes.c_double
    lib.spmm_tiles_time(32, ctypes.c_int64(M), ctypes.c_int64(K), ctypes.c_int64(N), ctypes.c_double(0), ctypes.c_double(0),
                        ctypes.byref(nb))
    return nb.value


def product(torch_gpu, csr, B, groups=4):  # noqa: F811
    """The product, of which the plan has to run in tiles of so many column groups."""
    assert column_groups(csr.M, csr.K, B.shape[1]) == groups
    C, plan = gpu_product(torch_gpu, csr, B, guard_rows=2, tiles=32)
    assert plan.describe()["tile_rows"] == 32
    return C


@pytest.mark.parametrize("M,K,N,density", [
    (64, 1, WIDE, 0.5), (33, 31, WIDE - 1, 1.0), (40, 257, WIDE - 5, 0.2), (64, 300, WIDE, 0.45), (64, 520, WIDE - 124, 0.7),
    (8192, 300, 100, 0.4), (8190, 545, 128, 1.0), (4090, 800, 200, 0.3), (9000, 64, 127, 0.6)])
def test_bit_exact_on_integer_data(torch_gpu, oracle, M, K, N, density):  # noqa: F811
    """Fewer steps than waves, odd and even numbers of them, rows, columns and steps cut short; blocks of one
    to four runs of 256 entries."""
    csr = integer_matrix(M, K, density, M + K)
    B = np.random.default_rng(N).integers(-16, 17, (K, N)).astype(np.float32)
    C = product(torch_gpu, csr, B)
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B, parallel=True)
    assert np.abs(C_ref).max() < 2 ** 24
    assert np.array_equal(C.astype(np.float64), C_ref)


@pytest.mark.parametrize("M,waves,groups", [(64, 8, 4), (32, 12, 2)])
def test_more_steps_than_a_run_of_bounds(torch_gpu, M, waves, groups):  # noqa: F811
    """65 steps and more per wave.  Integer data, compared on the device in 64 bits."""
    torch = torch_gpu
    K, N = 32 * waves * 65 + 40, WIDE
    assert column_groups(M, K, N) == groups
    csr = integer_matrix(M, K, 0.3, 3)
    dense = torch.zeros((M, K), device="cuda", dtype=torch.float64)
    rows = np.repeat(np.arange(M), np.diff(csr.row_ptr))
    dense[torch.from_numpy(rows).cuda(), torch.from_numpy(csr.col_idx).cuda().long()] = torch.from_numpy(csr.vals).cuda().double()
    B = torch.randint(-4, 5, (K, N), device="cuda", dtype=torch.int8).to(torch.float32)
    plan = spmm.plan_create(M, K, csr.row_ptr, csr.col_idx, csr.vals, tiles=32)
    C = plan.execute(B)
    for j in range(0, N, 2048):
        assert torch.equal(C[:, j:j + 2048].double(), dense @ B[:, j:j + 2048].double())


@pytest.mark.parametrize("M,K,N,density", [
    (32, 512, WIDE, 0.5), (32, 513, WIDE, 0.45), (31, 545, WIDE - 1, 1.0), (20, 800, WIDE // 2 + 8, 0.2), (32, 1300, WIDE - 70, 0.7),
    (8192, 600, 64, 0.3), (8190, 777, 63, 0.8), (4090, 800, 100, 0.6), (8192, 64, 50, 0.5)])
def test_two_column_groups(torch_gpu, oracle, M, K, N, density):  # noqa: F811
    """16 steps, which fp32 instructions multiply, and more: fewer than two per wave, remainders of waves, rows, columns
    and steps; blocks of one to four runs of 256 entries."""
    csr = integer_matrix(M, K, density, M + K)
    B = np.random.default_rng(N).integers(-16, 17, (K, N)).astype(np.float32)
    C = product(torch_gpu, csr, B, groups=2)
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B, parallel=True)
    assert np.abs(C_ref).max() < 2 ** 24
    assert np.array_equal(C.astype(np.float64), C_ref)


@pytest.mark.parametrize("a_scale,b_scale", [(1.0, 1.0), (1e-20, 1e10), (1.0, 1e-36), (1e-39, 1.0), (1e-10, 1e38), (1.0, None)])
def test_two_column_groups_with_every_part(torch_gpu, oracle, a_scale, b_scale):  # noqa: F811
    """The bounds of the two tests below, and a value outside the domain."""
    csr = few_entries(32, 600, 5, a_scale)
    B = np.random.default_rng(6).standard_normal((600, WIDE))
    if b_scale is None:
        B[::7] *= 1e-37
        B[csr.col_idx[3], 7] = np.inf
    else:
        B = (B * b_scale).clip(-3.4e38, 3.4e38)
    B = B.astype(np.float32)
    C = product(torch_gpu, csr, B, groups=2)
    C_ref, S = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, np.where(np.isinf(B), 0, B).astype(np.float32), parallel=True)
    fits = S < 3.4e38
    if b_scale is None:
        assert not np.isfinite(C[:, 7]).all()
        fits[:, 7] = False
    assert fits.mean() > 0.5
    assert (np.abs(C - C_ref)[fits] <= 2.0 ** -21 * S[fits] + 3 * 2.0 ** -149).all()


def few_entries(M, K, seed, scale):
    """Two entries in every row, one on its own in every eighth."""
    rng = np.random.default_rng(seed)
    W = np.zeros((M, K), np.float32)
    for i in range(M):
        n = 1 if i % 8 == 0 else 2
        W[i, rng.choice(K, n, replace=False)] = (rng.standard_normal(n) * scale).astype(np.float32)
    return gen.csr_from_dense(W)


@pytest.mark.parametrize("a_scale,b_scale", [(1.0, 1.0), (1e-20, 1e10), (1.0, 1e-36), (1e-36, 1.0), (1e-39, 1.0), (1.0, 1e-39), (1e-10, 1e38),
                                             (1e38, 1e-20)])
def test_every_part_of_a_product_counts(torch_gpu, oracle, a_scale, b_scale):  # noqa: F811
    """Sums of one or two products, so that nothing averages out.  Bound: a product's parts left out are below
    2^-24 of it, and there are at most twelve fp32 roundings, all but two of sums below 2^-7 of the result's terms: 2^-21.
    In the range of subnormal results add their spacing.  Values whose parts are not all normal (1e-36), subnormal ones and the largest."""
    csr = few_entries(64, 90, 5, a_scale)
    B = (np.random.default_rng(6).standard_normal((90, WIDE)) * b_scale).clip(-3.4e38, 3.4e38).astype(np.float32)
    B[3, :64] = np.float32(3.4028235e38) * min(1.0, b_scale)   # the largest float rounds up to no bf16
    C = product(torch_gpu, csr, B)
    C_ref, S = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B, parallel=True)
    fits = S < 3.4e38
    assert fits.mean() > 0.5
    assert (np.abs(C - C_ref)[fits] <= 2.0 ** -21 * S[fits] + 3 * 2.0 ** -149).all()


@pytest.mark.parametrize("M,groups", [(64, 4), (32, 2)])
def test_what_is_left_out_of_a_product(torch_gpu, oracle, M, groups):  # noqa: F811
    """One product per element, of the values that lose most.  m is at most 2^-8 and l 2^-17 of a value's leading bit, so
    m l + l m + l l are below 2^-24 of a product; adding the small sum rounds by 2^-24 once more, and its own five
    roundings, of sums below 2^-7, by less than 2^-27.  (With h cut off instead of rounded the first square loses 2^-22.02.)"""
    K, N = 600, WIDE
    near = np.concatenate([1 + 2.0 ** -7 - 2.0 ** -16 - np.arange(1, 9) * 2.0 ** -23, 1 + 2.0 ** -8 - 2.0 ** -17 + np.arange(-8, 9) * 2.0 ** -23,
                           1 + 2.0 ** -8 + 2.0 ** -17 + np.arange(-8, 9) * 2.0 ** -23, 1 + 3 * 2.0 ** -9 + np.arange(-8, 9) * 2.0 ** -23])
    rng = np.random.default_rng(M)
    W = np.zeros((M, K), np.float32)
    W[np.arange(M), rng.choice(K, M, replace=False)] = rng.choice(near, M) * rng.choice([-1, 1], M) * 2.0 ** rng.integers(-20, 20, M)
    csr = gen.csr_from_dense(W)
    B = (rng.choice(near, (K, N)) * rng.choice([-1, 1], (K, N))).astype(np.float32)
    C = product(torch_gpu, csr, B, groups)
    C_ref, S = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B, parallel=True)
    assert (np.abs(C - C_ref) <= (2.0 ** -23 + 2.0 ** -27) * S).all()


def test_a_few_tiny_values_among_ordinary_ones(torch_gpu, oracle):  # noqa: F811
    csr = few_entries(64, 300, 7, 1.0)
    B = np.random.default_rng(8).standard_normal((300, WIDE)).astype(np.float32)
    B[::7] *= np.float32(1e-37)
    C = product(torch_gpu, csr, B)
    C_ref, S = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B, parallel=True)
    assert (np.abs(C - C_ref) <= 2.0 ** -21 * S + 3 * 2.0 ** -149).all()


@pytest.mark.parametrize("M,groups", [(64, 4), (32, 2)])
@pytest.mark.parametrize("exponents,power", [((-112, -108), 2.0 ** 40), ((126, 127), 2.0 ** -20)])
@pytest.mark.parametrize("of_a", [False, True])
def test_ends_of_the_range_of_parts(torch_gpu, M, groups, exponents, power, of_a):  # noqa: F811
    """Values around 2^-110, below which the last part is no bf16, and around 2^128 - 2^119, from which the first is infinite, times a
    power of two: every value is the sum of its parts or multiplied in fp32, so each product is exact."""
    K, N = 600, WIDE
    rng = np.random.default_rng(M)

    def ends(shape):
        mantissa = np.where(rng.random(shape) < 0.5, rng.integers(0, 1 << 23, shape), (1 << 23) - rng.choice([1, 2, 3, 1 << 14, (1 << 14) + 1, (1 << 15) + 1], shape))
        return (np.ldexp(1 + mantissa * 2.0 ** -23, rng.integers(exponents[0], exponents[1] + 1, shape)) * rng.choice([-1, 1], shape)).astype(np.float32)

    W = np.zeros((M, K), np.float32)
    columns = rng.choice(K, M, replace=False)
    W[np.arange(M), columns] = ends(M) if of_a else power
    B = np.full((K, N), power, np.float32) if of_a else ends((K, N))
    C = product(torch_gpu, gen.csr_from_dense(W), B, groups)
    assert np.isfinite(C).all()
    assert np.array_equal(C, W[np.arange(M), columns][:, None] * B[columns])


def with_tails(rng, K, N, share):
    """Normal values, some so small that they are no sum of three bf16 numbers, subnormal ones among them."""
    B = rng.standard_normal((K, N)).astype(np.float32)
    tiny = rng.random((K, N)) < share
    B[tiny] *= 10.0 ** rng.uniform(-44, -34, int(tiny.sum())).astype(np.float32)
    return B


@pytest.mark.parametrize("share", [0.01, 0.6, 1.0])
@pytest.mark.parametrize("M,K,N,groups", [(64, 600, WIDE, 4), (57, 300, WIDE - 5, 4), (32, 1300, WIDE // 2 + 6, 2)])
@pytest.mark.parametrize("tiny_in_a", [False, True])
def test_tails(torch_gpu, oracle, M, K, N, groups, share, tiny_in_a):  # noqa: F811
    """Whether a wave takes its first or its second result: columns with and without ordinary values, columns of zeros and tiny ones, rows
    without entries (of the matrix, of a wave), columns past the last, and values of A that are no such sum.  Bound: 2^-24 of
    what is left out of a product, and fewer than 120 roundings, one per 16 columns of A (two with fp32 instructions) and wave."""
    rng = np.random.default_rng(K + N)
    W = np.where(rng.random((M, K)) < 0.4, rng.standard_normal((M, K)), 0.0).astype(np.float32)
    W[5] = 0
    W[9, 1:] = 0
    W[11, : K // 2] = 0
    if tiny_in_a:
        W[3, 7] = 1e-40
        W[20, 50:60] = 3e-36
    csr = gen.csr_from_dense(W)
    B = with_tails(rng, K, N, share)
    B[:, 3] = 0
    B[:, 17] = np.where(np.arange(K) % 3 == 0, 1e-40, 0)
    B[:, N - 1] = 2e-38
    C = product(torch_gpu, csr, B, groups)
    C_ref, S = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B, parallel=True)
    steps = (K + 31) // 32
    assert (np.abs(C - C_ref) <= (steps * 16 + 40) * 2.0 ** -24 * S + steps * 16 * 2.0 ** -149).all()


@pytest.mark.parametrize("M,K,sparsity,groups", [(8192, 2048, 0.5, 4), (4096, 4096, 0.5, 2), (4096, 1024, 0.97, 2)])
def test_tails_take_no_second_pass(torch_gpu, M, K, sparsity, groups):  # noqa: F811
    """Values that cannot change a result cost no time.  (With a second pass for each of them the product takes 2.7 times as long.)"""
    torch = torch_gpu
    csr = gen.uniform_positions(M, K, sparsity, 3)
    plan = spmm.plan_create(csr.M, K, csr.row_ptr, csr.col_idx, csr.vals, tiles=32)
    rng = np.random.default_rng(1)
    ordinary, tails = (torch.from_numpy(with_tails(rng, K, 128, share)).cuda() for share in (0.0, 0.05))
    C = torch.empty((csr.M, 128), device="cuda")

    def fastest(B):
        times = []
        for _ in range(8):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            for _ in range(20):
                plan.execute(B, C)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    assert column_groups(M, K, 128) == groups
    fastest(ordinary)
    assert fastest(tails) < 1.5 * fastest(ordinary)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_how_far_a_value_outside_the_domain_reaches(torch_gpu, value):  # noqa: F811
    """As on the other tiles: its column of C and no other."""
    csr = gen.uniform_positions(64, 256, 0.5, 15)
    B = gen.dense_activations(csr.K, WIDE, 16)
    B[100, 7] = value
    C = product(torch_gpu, csr, B)
    finite = np.isfinite(C)
    assert not finite[:, 7].any() and np.delete(finite, 7, axis=1).all()
