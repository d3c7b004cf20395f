"""Matrix-core path (spmm_options_t.tiles) against the CPU oracle, through the C ABI (needs the GPU)."""
import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen

from test_gpu_parity import check, gpu_product, torch_gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def integer_matrix(M, K, density, seed):
    rng = np.random.default_rng(seed)
    W = np.where(rng.random((M, K)) < density, rng.integers(-8, 9, (M, K)), 0).astype(np.float32)
    W[min(5, M - 1)] = rng.integers(1, 9, K)   # a dense row
    W[M // 2] = 0                              # an empty one
    return gen.csr_from_dense(W)


@pytest.mark.parametrize("N", [1, 3, 16, 17, 32, 33, 64, 100, 128, 129, 300])
@pytest.mark.parametrize("tiles", [16, 32])
@pytest.mark.parametrize("M,K", [(3, 1), (15, 65), (33, 511), (70, 1024), (257, 2050)])
def test_tiles_are_bit_exact_on_integer_data(torch_gpu, oracle, M, K, tiles, N):  # noqa: F811
    """Panels, column steps and column tiles that do not divide the sizes, fewer steps than waves
    and more, dense and empty rows; any order of the sums is exact."""
    csr = integer_matrix(M, K, 0.4, M + K)
    B = np.random.default_rng(N).integers(-16, 17, (K, N)).astype(np.float32)
    C, plan = gpu_product(torch_gpu, csr, B, guard_rows=2, tiles=tiles)
    assert plan.describe()["tile_rows"] == tiles
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B)
    assert np.abs(C_ref).max() < 2 ** 24
    assert np.array_equal(C.astype(np.float64), C_ref)


@pytest.mark.parametrize("N", [20, 64, 128])
@pytest.mark.parametrize("M,K,tiles", [(4096, 300, 16), (4096, 300, 32), (8192, 520, 32)])
def test_tiles_with_workgroups_for_the_whole_chip(torch_gpu, oracle, M, K, tiles, N):  # noqa: F811
    """Panels enough that the wider column tiles are taken; real values."""
    csr = gen.lognormal_rows(M, K, 0.6, 7)
    B = gen.dense_activations(K, N, 8)
    C, plan = gpu_product(torch_gpu, csr, B, guard_rows=1, tiles=tiles)
    assert plan.describe()["tile_rows"] == tiles
    check(oracle, csr, B, C, parallel=True)


def test_tiles_chosen_by_density_and_left_alone_by_other_settings(torch_gpu, oracle):  # noqa: F811
    dense, sparse = gen.uniform_positions(2048, 2048, 0.6, 1), gen.uniform_positions(2048, 2048, 0.95, 2)
    B = gen.dense_activations(2048, 128, 3)
    C, plan = gpu_product(torch_gpu, dense, B, n_hint=128)
    assert plan.describe()["tile_rows"] > 0 and plan.describe()["scratch_bytes"] == 0
    check(oracle, dense, B, C, parallel=True)
    for kw in (dict(tiles=-1), dict(ufi=8), dict(kslices=2), dict(sort_rows=1)):
        assert gpu_product(torch_gpu, dense, B, n_hint=128, **kw)[1].describe()["tile_rows"] == 0
    assert gpu_product(torch_gpu, sparse, B, n_hint=128)[1].describe()["tile_rows"] == 0


def test_tiles_with_unsorted_columns_duplicates_and_bad_columns(torch_gpu, oracle):  # noqa: F811
    """The order of a row's entries does not matter (bit for bit); a column stored twice keeps the
    matrix on chunks; a column outside A is refused."""
    csr = gen.uniform_positions(90, 700, 0.5, 4)
    rng = np.random.default_rng(5)
    rows = np.repeat(np.arange(csr.M), np.diff(csr.row_ptr))
    o = np.lexsort((rng.random(len(rows)), rows))
    B = gen.dense_activations(csr.K, 50, 6)
    C0, _ = gpu_product(torch_gpu, csr, B, tiles=16)
    C1, plan = gpu_product(torch_gpu, gen.Csr(csr.M, csr.K, csr.row_ptr, csr.col_idx[o], csr.vals[o]), B, tiles=16)
    assert plan.describe()["tile_rows"] == 16 and np.array_equal(C0, C1)
    check(oracle, csr, B, C1)
    twice = csr.col_idx.copy()
    twice[1] = twice[0]
    csr2 = gen.Csr(csr.M, csr.K, csr.row_ptr, twice, csr.vals)
    C2, plan = gpu_product(torch_gpu, csr2, B, tiles=16)
    assert plan.describe()["tile_rows"] == 0
    check(oracle, csr2, B, C2)
    for bad in (-1, csr.K):
        col = csr.col_idx.copy()
        col[100] = bad
        with pytest.raises(spmm.SpmmError) as err:
            spmm.plan_create(csr.M, csr.K, csr.row_ptr, col, csr.vals, tiles=16)
        assert err.value.status == spmm.SPMM_ERR_INVALID_CSR


@pytest.mark.parametrize("tiles", [16, 32])
def test_tiles_with_rows_of_b_too_long_for_32_bit_offsets(torch_gpu, oracle, tiles):  # noqa: F811
    """A step's rows of B span more than 4 GiB: 64-bit addresses.  Checked on columns at both ends."""
    torch = torch_gpu
    csr = integer_matrix(20, 33, 0.5, 9)
    N = (1 << 32) // (1024 // tiles * 4) + 3
    B = torch.randint(-9, 10, (csr.K, N), device="cuda", dtype=torch.int8).to(torch.float32)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=tiles)
    assert plan.describe()["tile_rows"] == tiles
    C = plan.execute(B)
    cols = torch.cat([torch.arange(0, 200), torch.arange(N - 200, N)]).cuda()
    B_small, C_small = B[:, cols].contiguous().cpu().numpy(), C[:, cols].cpu().numpy()
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B_small)
    assert np.array_equal(C_small.astype(np.float64), C_ref)


def test_tiles_replay_from_a_graph_and_overlap_on_streams(torch_gpu, oracle):  # noqa: F811
    torch = torch_gpu
    csr = gen.uniform_positions(300, 900, 0.5, 11)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=16)
    B = torch.from_numpy(gen.dense_activations(csr.K, 64, 12)).cuda()
    C = torch.full((csr.M, 64), float("nan"), device="cuda")
    eager = plan.execute(B).clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        outs = [plan.execute(B) for _ in range(3)]
    here = [plan.execute(B) for _ in range(3)]
    torch.cuda.synchronize()
    assert all(torch.equal(x, eager) for x in outs + here)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.execute(B, C)
    for _ in range(3):
        C.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, eager)
        plan.execute(B)
        torch.cuda.synchronize()
    check(oracle, csr, B.cpu().numpy(), eager.cpu().numpy())


@pytest.mark.parametrize("tiles", [16, 32])
def test_as_many_columns_as_the_interface_counts(torch_gpu, tiles):  # noqa: F811
    """N = 2^31 - 1: the number of column tiles is rounded up beyond 31 bits.  One row of A, so that
    C is a sum of scaled rows of B; all of it is compared, a run of columns at a time."""
    torch = torch_gpu
    N = 2 ** 31 - 1
    plan = spmm.plan_create(1, 2, np.array([0, 2]), np.array([0, 1]), np.array([3.0, -2.0]), tiles=tiles)
    assert plan.describe()["tile_rows"] == tiles
    B = torch.empty((2, N), device="cuda")
    for j in range(0, N, 1 << 28):
        B[:, j:j + (1 << 28)] = torch.randint(-9, 10, B[:, j:j + (1 << 28)].shape, device="cuda", dtype=torch.int8)
    C = plan.execute(B)
    for j in range(0, N, 1 << 28):
        assert torch.equal(C[0, j:j + (1 << 28)], 3 * B[0, j:j + (1 << 28)] - 2 * B[1, j:j + (1 << 28)]), j


def test_more_rows_than_a_launch_of_the_builder_takes(torch_gpu):  # noqa: F811
    """2^26 rows, one wave each, are one launch more than HIP takes: the matrix stays on chunks."""
    torch = torch_gpu
    M = (1 << 26) + 8
    row_ptr = (np.arange(M + 1) + 63) // 64          # every 64th row has an entry
    nnz = int(row_ptr[-1])
    vals = (np.arange(nnz) % 64 - 31).astype(np.float32)
    plan = spmm.plan_create(M, 1, row_ptr, np.zeros(nnz), vals, tiles=8)
    assert plan.describe()["tile_rows"] == 0
    C = plan.execute(torch.full((1, 1), 3.0, device="cuda"))
    want = torch.zeros(M, device="cuda")
    want[::64] = 3 * torch.from_numpy(vals).cuda()
    assert torch.equal(C[:, 0], want)


def test_a_plan_is_created_while_another_stream_works(torch_gpu, oracle):  # noqa: F811
    """Building tiles waits for the builder's own work only, and its working memory goes back to the device."""
    torch = torch_gpu
    csr = gen.uniform_positions(1024, 1024, 0.5, 13)
    B = gen.dense_activations(csr.K, 64, 14)
    C, plan = gpu_product(torch, csr, B, tiles=16)   # everything is loaded
    plan.destroy()
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)   # its first call also loads the kernel
    torch.cuda.synchronize()
    start.record()
    torch.cuda._sleep(1000000)
    end.record()
    torch.cuda.synchronize()
    cycles = int(1000000 * 200.0 / start.elapsed_time(end))   # 200 ms
    for _ in range(8):   # a stream that shares the builder's hardware queue (one of four) holds it up whatever the library does
        side, done = torch.cuda.Stream(), torch.cuda.Event()
        with torch.cuda.stream(side):
            torch.cuda._sleep(1000)
            torch.cuda.synchronize()
            free = torch.cuda.mem_get_info()[0]
            torch.cuda._sleep(cycles)
            done.record()
        plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=16)
        waited = done.query()
        if not waited:
            break
        plan.destroy()
    assert not waited, "the creation waited for the other stream"
    assert plan.describe()["tile_rows"] == 16
    assert free - torch.cuda.mem_get_info()[0] <= plan.describe()["device_bytes"] + (4 << 20)
    dC = plan.execute(torch.from_numpy(B).cuda())
    assert np.array_equal(dC.cpu().numpy(), C)
    check(oracle, csr, B, C)
    side.synchronize()


def test_how_far_a_value_outside_the_domain_reaches(torch_gpu):  # noqa: F811
    """B is finite by contract.  An infinity in one row of it stays in its column of C on both paths, and on
    single rows of chunks in the rows with an entry there (and in none that has no entry in its chunks)."""
    torch = torch_gpu
    csr = gen.uniform_positions(64, 256, 0.5, 15)
    B = gen.dense_activations(csr.K, 32, 16)
    k, j = 100, 7
    B[k, j] = np.inf
    dense = np.zeros((csr.M, csr.K), np.float32)
    dense[np.repeat(np.arange(csr.M), np.diff(csr.row_ptr)), csr.col_idx] = csr.vals
    holds = dense[:, k] != 0
    for tiles in (-1, 8, 16, 32):
        C, _ = gpu_product(torch, csr, B, tiles=tiles, ufi=1 if tiles < 0 else 0)
        finite = np.isfinite(C)
        assert finite[:, [c for c in range(32) if c != j]].all()
        assert not finite[holds, j].any()
        assert finite[~holds, j].all() if tiles < 0 else not finite[:, j].any()


@pytest.mark.parametrize("N", [1, 4, 36, 128, 1000, 4099])
@pytest.mark.parametrize("tiles,n_hint", [(8, 4), (8, 16), (16, 64), (32, 128)])
def test_tile_plans_at_widths_far_from_their_hint(torch_gpu, oracle, tiles, n_hint, N):  # noqa: F811
    """A plan stays valid for every N: fewer columns than a column group, and many column tiles (more
    workgroups than the chip holds at once, in several XCD shares)."""
    csr = integer_matrix(530, 700, 0.3, 17)
    B = np.random.default_rng(N).integers(-16, 17, (csr.K, N)).astype(np.float32)
    C, plan = gpu_product(torch_gpu, csr, B, guard_rows=2, tiles=tiles, n_hint=n_hint)
    assert plan.describe()["tile_rows"] == tiles
    C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, B)
    assert np.array_equal(C.astype(np.float64), C_ref)


@pytest.mark.parametrize("tiles", [8, 16, 32])
def test_tile_plans_with_operands_at_4_byte_offsets(torch_gpu, oracle, tiles):  # noqa: F811
    """The interface asks for 4-byte alignment only; nothing beside C is written, through either entry point."""
    torch = torch_gpu
    csr = integer_matrix(75, 300, 0.4, 19)
    plan = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=tiles)
    for N in (4, 8, 16, 64, 130):
        Bh = np.random.default_rng(N).integers(-16, 17, (csr.K, N)).astype(np.float32)
        C_ref, _ = oracle.spmm(csr.row_ptr, csr.col_idx, csr.vals, Bh)
        for offset in (1, 2, 3):
            memory = torch.full((csr.K * N + 8,), float("nan"), device="cuda")
            B = memory[offset:offset + csr.K * N].view(csr.K, N)
            B.copy_(torch.from_numpy(Bh))
            for run in (plan.execute_raw, plan.execute_static_raw):
                out = torch.full((csr.M * N + 8,), float("nan"), device="cuda")
                run(B.data_ptr(), N, out.data_ptr() + 4 * offset, None)
                torch.cuda.synchronize()
                host = out.cpu().numpy()
                assert np.array_equal(host[offset:offset + csr.M * N].reshape(csr.M, N).astype(np.float64), C_ref)
                assert np.isnan(host[:offset]).all() and np.isnan(host[offset + csr.M * N:]).all()
    for bad in (1, 2):
        with pytest.raises(spmm.SpmmError) as err:
            plan.execute_raw(B.data_ptr() + bad, N, out.data_ptr(), None)
        assert err.value.status == spmm.SPMM_ERR_INVALID_ARG


def test_values_of_the_tiles_setting(torch_gpu):  # noqa: F811
    csr = gen.uniform_positions(40, 60, 0.5, 21)
    for bad in (1, 4, 12, 24, 33, 64, 2 ** 31 - 1):
        with pytest.raises(spmm.SpmmError) as err:
            spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=bad)
        assert err.value.status == spmm.SPMM_ERR_INVALID_ARG
    for off in (-1, -8, -2 ** 31):
        assert spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=off).describe()["tile_rows"] == 0
    host = spmm.plan_create(csr.M, csr.K, csr.row_ptr, csr.col_idx, csr.vals, tiles=16, host_only=True)
    assert host.describe()["tile_rows"] == 0
    empty = spmm.plan_create(40, 60, np.zeros(41), [], [], tiles=16)   # no entry at all
    B = torch_gpu.ones((60, 8), device="cuda")
    assert torch_gpu.equal(empty.execute(B), torch_gpu.zeros((40, 8), device="cuda"))
