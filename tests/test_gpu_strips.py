"""The strips path (eight columns of B in LDS, one lane per part of a row) against the oracle, at the edges of its units, bands
and strips.  Needs the GPU."""
import ctypes

import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen
from test_gpu_parity import check, gpu_product, torch_gpu  # noqa: F401
from test_gpu_tiles import integer_matrix

pytestmark = pytest.mark.gpu


def strips_of(csr, n_hint):
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, n_hint=n_hint, strips=1)
    info = plan.describe()
    assert info["strip_units"] > 0 and info["tile_rows"] == 0 and info["scratch_bytes"] == 0
    return plan


@pytest.mark.parametrize("N", [1, 7, 8, 9, 64, 130, 4099])
@pytest.mark.parametrize("M,K,density,hint", [(2, 3, 0.9, 8), (2, 5000, 0.99, 200), (65, 100, 0.2, 16), (257, 5088, 0.1, 0), (257, 5089, 0.1, 64),
                                              (70, 11000, 0.05, 128), (1500, 300, 0.02, 256)])
def test_whole_numbers_are_exact(torch_gpu, oracle, M, K, density, hint, N):  # noqa: F811
    """Rows in 1 to 64 parts, strips in one to three bands, few and many columns of B; B and C at every
    offset that the interface allows, nothing beside C written, through both entry points."""
    torch = torch_gpu
    csr = integer_matrix(M, K, density, 5)
    plan = strips_of(csr, hint)
    Bh = np.random.default_rng(N).integers(-16, 17, (K, N)).astype(np.float32)
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, Bh)
    for offset, run in ((0, plan.execute_raw), (1, plan.execute_static_raw), (3, plan.execute_raw)):
        memory = torch.full((K * N + 8,), float("nan"), device="cuda")
        B = memory[offset:offset + K * N].view(K, N)
        B.copy_(torch.from_numpy(Bh))
        out = torch.full((M * N + 8,), float("nan"), device="cuda")
        run(B.data_ptr(), N, out.data_ptr() + 4 * offset, None)
        torch.cuda.synchronize()
        host = out.cpu().numpy()
        assert np.array_equal(host[offset:offset + M * N].reshape(M, N).astype(np.float64), C_ref)
        assert np.isnan(host[:offset]).all() and np.isnan(host[offset + M * N:]).all()


@pytest.mark.parametrize("make,M,K,sparsity,N", [(gen.uniform_positions, 4096, 4096, 0.95, 128), (gen.lognormal_rows, 3001, 2511, 0.85, 200),
                                                 (gen.zipf_rows, 2000, 9000, 0.93, 60), (gen.zipf_rows, 3000, 700, 0.8, 33), (gen.lognormal_rows, 9000, 400, 0.7, 20)])
def test_against_the_oracle(torch_gpu, oracle, make, M, K, sparsity, N):  # noqa: F811
    csr = make(M, K, sparsity, 6)
    B = gen.dense_activations(K, N, 7)
    C, plan = gpu_product(torch_gpu, csr, B, guard_rows=2, n_hint=N, strips=1)
    assert plan.describe()["strip_units"] > 0
    check(oracle, csr, B, C, parallel=True)
    C2, _ = gpu_product(torch_gpu, csr, B, n_hint=N, strips=1, threads=3)
    assert np.array_equal(C, C2)


@pytest.mark.parametrize("make,M,K,sparsity,hint", [(gen.lognormal_rows, 300, 6000, 0.97, 40), (gen.zipf_rows, 1000, 700, 0.8, 0), (gen.zipf_rows, 5, 12000, 0.6, 8),
                                                    (gen.uniform_positions, 3000, 1000, 0.75, 200), (gen.lognormal_rows, 700, 9001, 0.9, 16)])
def test_the_builders_on_the_device_and_on_the_host_agree(torch_gpu, make, M, K, sparsity, hint):  # noqa: F811
    """The order of a row's entries does not matter, bit for bit: where they are in order of the columns, the strips
    are built on the device, else on the host; both make the same words."""
    rng = np.random.default_rng(8)
    csr = make(M, K, sparsity, 9)
    order = np.concatenate([rng.permutation(np.arange(a, b)) for a, b in zip(csr.row_ptr[:-1], csr.row_ptr[1:])])
    B = gen.dense_activations(K, 40, 10)
    C0, one = gpu_product(torch_gpu, csr, B, strips=1, n_hint=hint)
    C1, two = gpu_product(torch_gpu, gen.Csr(M, K, csr.row_ptr, csr.col_idx[order], csr.vals[order]), B, strips=1, n_hint=hint)
    assert np.array_equal(C0, C1) and one.describe() == two.describe()
    same_strips(one, two)
    # out of order only at the end of a long row: the device finds it and the host builds
    end = csr.row_ptr[np.argmax(np.diff(csr.row_ptr)) + 1]
    order = np.arange(csr.row_ptr[-1])
    order[end - 2:end] = order[end - 2:end][::-1]
    C2, three = gpu_product(torch_gpu, gen.Csr(M, K, csr.row_ptr, csr.col_idx[order], csr.vals[order]), B, strips=1, n_hint=hint)
    assert np.array_equal(C0, C2)
    same_strips(one, three)


def words(plan):
    """The words of a plan on strips, and whether they were made on the device."""
    lib = ctypes.CDLL(spmm.load()._name)
    lib.spmm_strips_words.restype = ctypes.c_int64
    on_device = ctypes.c_int32(-1)
    n = lib.spmm_strips_words(plan.handle, None, ctypes.c_int64(0), ctypes.byref(on_device))
    out = np.zeros(n, np.uint32)
    assert n > 0 and lib.spmm_strips_words(plan.handle, ctypes.c_void_p(out.ctypes.data), ctypes.c_int64(n), None) == n
    return out, on_device.value


def same_strips(by_device, by_host):
    (one, on_device), (two, on_host) = words(by_device), words(by_host)
    assert (on_device, on_host) == (1, 0) and np.array_equal(one, two)


def in_order(nnz, K, seed):
    """64 rows, in all `nnz` entries, columns in order."""
    rng = np.random.default_rng(seed)
    lens = np.full(64, nnz // 64)
    lens[:nnz - lens.sum()] += 1
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col_idx = np.concatenate([np.sort(rng.permutation(K)[:n]) for n in lens]).astype(np.int32)
    return row_ptr, col_idx, rng.integers(-8, 9, nnz).astype(np.float32)


# columns of 16 bits and, from 65537 on, of 32; from ordinary memory and through pinned memory, in one piece or several
@pytest.mark.parametrize("nnz,K", [((1 << 19) - 1, 70000), (1 << 19, 20000), ((1 << 19) + 1, 65536), ((1 << 19) + 1, 65537), (2200003, 65536), (3500001, 70000)])
def test_large_matrices_reach_the_device_whole(torch_gpu, nnz, K):  # noqa: F811
    torch = torch_gpu
    row_ptr, col_idx, vals = in_order(nnz, K, nnz % 1000)
    plan = spmm.plan_create(64, K, row_ptr, col_idx, vals, strips=1)
    B = torch.randint(-4, 5, (K, 4), device="cuda", dtype=torch.int8).to(torch.float32)
    rows = torch.from_numpy(np.repeat(np.arange(64), np.diff(row_ptr))).cuda()
    terms = torch.from_numpy(vals).cuda().double()[:, None] * B[torch.from_numpy(col_idx).cuda().long()].double()
    assert torch.equal(plan.execute(B).double(), torch.zeros((64, 4), device="cuda", dtype=torch.float64).index_add_(0, rows, terms))
    order = np.concatenate([np.arange(a, b)[::-1] for a, b in zip(row_ptr[:-1], row_ptr[1:])])
    same_strips(plan, spmm.plan_create(64, K, row_ptr, col_idx[order], vals[order], strips=1))


@pytest.mark.parametrize("nnz,K", [(2200003, 40000), (2200003, 70000), (9000, 70000)])
def test_columns_outside_are_found_on_the_device(torch_gpu, nnz, K):  # noqa: F811
    """In the first, the middle and the last piece of the upload; in rows that are otherwise in order."""
    row_ptr, col_idx, vals = in_order(nnz, K, 1)
    for row in (0, 31, 63):
        for at, outside in ((row_ptr[row], -1), (row_ptr[row + 1] - 1, K), (row_ptr[row + 1] - 1, 2 ** 31 - 1), (row_ptr[row], -65536), (row_ptr[row + 1] - 1, K + 65536)):
            bad = col_idx.copy()
            bad[at] = outside
            with pytest.raises(spmm.SpmmError) as err:
                spmm.plan_create(64, K, row_ptr, bad, vals, strips=1)
            assert err.value.status == spmm.SPMM_ERR_INVALID_CSR
    assert words(spmm.plan_create(64, K, row_ptr, col_idx, vals, strips=1))[1] == 1   # the memory was given back


def test_duplicates_empty_rows_and_bad_columns(torch_gpu, oracle):  # noqa: F811
    """Duplicates are summed, in any order and side by side; a column outside A is refused."""
    rng = np.random.default_rng(8)
    B = gen.dense_activations(300, 40, 10)
    lens = rng.integers(0, 90, 200)
    lens[::7] = 0
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    csr = gen.Csr(200, 300, row_ptr, rng.integers(0, 300, row_ptr[-1]).astype(np.int32), rng.standard_normal(row_ptr[-1]).astype(np.float32))
    in_order = np.concatenate([np.sort(csr.col_idx[a:b]) for a, b in zip(row_ptr[:-1], row_ptr[1:])])
    for a in (csr, gen.Csr(200, 300, row_ptr, in_order, csr.vals)):
        C, _ = gpu_product(torch_gpu, a, B, guard_rows=1, strips=1)
        check(oracle, a, B, C)
    for bad in (-1, 300):
        col = csr.col_idx.copy()
        col[-1] = bad
        with pytest.raises(spmm.SpmmError) as err:
            spmm.plan_create(200, 300, row_ptr, col, csr.vals, strips=1)
        assert err.value.status == spmm.SPMM_ERR_INVALID_CSR


@pytest.mark.parametrize("K", [4096, 16384])
def test_what_the_builder_worked_with_is_given_back(torch_gpu, K):  # noqa: F811
    """When the creation returns, not with the next synchronisation; with one band and with four."""
    torch = torch_gpu
    csr = gen.uniform_positions(8192, K, 0.96, 3)
    strips_of(csr, 64)   # what the runtime sets up once
    torch.cuda.synchronize()
    plan = strips_of(csr, 64)
    free = torch.cuda.mem_get_info()[0]
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free and plan.describe()["n_chunks"] == plan.describe()["strip_units"] * (1 if K == 4096 else 4)


def test_no_chain_of_additions_is_longer_than_twelve_groups(torch_gpu):  # noqa: F811
    """A row of 2^24 and ones, two of a lane in each of 30 bands, a group each: the chain of the 2^24 loses every one that it meets.  It meets eleven
    at most, and the sums of the parts of a row, rounded to even numbers, are off by one in each of six additions."""
    torch, bands = torch_gpu, 30
    K, in_band = bands * 5088, 128
    col = np.concatenate([b * 5088 + np.arange(in_band) for b in range(bands)]).astype(np.int32)
    for big in (0, 1, 77):
        vals = np.ones(col.size, np.float32)
        vals[big] = 2.0 ** 24
        plan = spmm.plan_create(1, K, np.array([0, col.size]), col, vals, strips=1)
        assert plan.describe()["n_chunks"] == bands and plan.describe()["n_enum"] == bands * 64 * 4
        C = plan.execute(torch.ones((K, 8), device="cuda"))
        off = (C.double() - (2.0 ** 24 + col.size - 1)).abs()
        assert float(off.max()) <= 11 + 6


def test_a_value_outside_the_domain_reaches_only_rows_with_an_entry_there(torch_gpu):  # noqa: F811
    csr = gen.uniform_positions(64, 256, 0.5, 15)
    B = gen.dense_activations(csr.K, 32, 16)
    B[100, 7] = np.inf
    holds = np.zeros(csr.M, bool)
    holds[np.repeat(np.arange(csr.M), np.diff(csr.row_ptr))[csr.col_idx == 100]] = True
    C, _ = gpu_product(torch_gpu, csr, B, strips=1)
    finite = np.isfinite(C)
    assert not finite[holds, 7].any() and finite[~holds].all() and finite[:, [c for c in range(32) if c != 7]].all()


def test_more_workgroups_than_a_launch_takes_and_addresses_beyond_32_bits(torch_gpu):  # noqa: F811
    """33.6 million columns of B: 4.2 million strips (a launch takes 4.19 million workgroups of 1024 threads) and rows of 134 MB, of which 32
    span more than 4 GiB."""
    torch, N = torch_gpu, (1 << 25) + 9
    plan = spmm.plan_create(2, 3, np.array([0, 2, 3]), np.array([0, 2, 1]), np.array([3.0, -2.0, 5.0]), strips=1)
    assert plan.describe()["strip_units"] > 0
    B = torch.randint(-9, 10, (3, N), device="cuda").float()
    C = plan.execute(B)
    assert torch.equal(C[0], 3 * B[0] - 2 * B[2]) and torch.equal(C[1], 5 * B[1])


def test_when_strips_are_chosen(torch_gpu):  # noqa: F811
    """Where chunks would gather slowly and tiles would multiply too many zeros; never with another setting, never against one."""
    csr = gen.uniform_positions(4096, 4096, 0.95, 1)
    args = (csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals)
    assert spmm.plan_create(*args, n_hint=128).describe()["strip_units"] > 0
    for kw in (dict(tiles=-1), dict(strips=-1), dict(ufi=4), dict(kslices=2), dict(tiles=16)):
        assert spmm.plan_create(*args, n_hint=128, **kw).describe()["strip_units"] == 0
    for kw in (dict(ufi=4), dict(host_only=True), dict(force_wide=True)):
        with pytest.raises(spmm.SpmmError) as err:
            spmm.plan_create(*args, strips=1, **kw)
        assert err.value.status == spmm.SPMM_ERR_INVALID_ARG
    # instead of tiles of 16 rows, but neither of 8 rows nor of the wide ones of 32; from rows out of order the tiles stay
    csr = gen.uniform_positions(4096, 2048, 0.8, 2)
    for n_hint, rows in ((64, 0), (4, 8)):
        info = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, n_hint=n_hint).describe()
        assert info["tile_rows"] == rows and (info["strip_units"] > 0) == (rows == 0)
    csr.col_idx[:2] = csr.col_idx[1::-1]
    assert spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, n_hint=64).describe()["tile_rows"] == 16
    # not where the rows' entries lie together, so that most lanes wait in most bands of columns
    for apart in (True, False):
        csr = gen.uniform_positions(2048, 16384 if apart else 4096, 0.9 if apart else 0.6, 4)
        if not apart:
            csr = gen.Csr(2048, 16384, csr.row_ptr, csr.col_idx + 4096 * np.repeat(np.arange(2048) * 7919 % 4, np.diff(csr.row_ptr)).astype(np.int32), csr.vals)
        info = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, n_hint=200).describe()
        assert info["tile_rows"] == 0 and (info["strip_units"] > 0) == apart
    csr = gen.uniform_positions(2048, 4096, 0.5, 3)
    assert spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, n_hint=256).describe()["tile_rows"] == 32
    assert spmm.plan_create(40, 60, np.zeros(41), [], [], strips=1).describe()["strip_units"] == 0   # no entry at all
