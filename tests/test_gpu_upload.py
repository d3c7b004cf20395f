"""Plans on tiles whose arrays go to the device through pinned memory (needs the GPU)."""
import gc
import threading

import numpy as np
import pytest

import paper_2506_15174_amd as spmm

from test_gpu_parity import torch_gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SMALLEST = 1 << 19   # entries


def matrix(nnz, K, seed):
    """64 rows, of lengths that differ, in all `nnz` entries; columns in no order."""
    rng = np.random.default_rng(seed)
    lens = np.full(64, nnz // 64)
    lens[:nnz - lens.sum()] += 1
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col_idx = np.concatenate([rng.permutation(K)[:n] for n in lens]).astype(np.int32)
    return row_ptr, col_idx, rng.integers(-8, 9, nnz).astype(np.float32)


def right(torch, plan, K, row_ptr, col_idx, vals):
    B = torch.randint(-4, 5, (K, 4), device="cuda", dtype=torch.int8).to(torch.float32)
    rows = torch.from_numpy(np.repeat(np.arange(64), np.diff(row_ptr))).cuda()
    terms = torch.from_numpy(vals).cuda().double()[:, None] * B[torch.from_numpy(col_idx).cuda().long()].double()
    return torch.equal(plan.execute(B).double(), torch.zeros((64, 4), device="cuda", dtype=torch.float64).index_add_(0, rows, terms))


# columns of 16 bits and, from 65537 on, of 32; one piece of memory or several, and more than it holds at once
@pytest.mark.parametrize("nnz,K", [(SMALLEST - 1, 20000), (SMALLEST, 20000), (SMALLEST + 1, 65536), (SMALLEST + 1, 65537), ((1 << 21) + 17, 65536),
                                   (3500001, 65537), (4100000, 65536), (7000003, 200000)])
def test_every_entry_arrives(torch_gpu, nnz, K):  # noqa: F811
    arrays = matrix(nnz, K, nnz % 1000)
    plan = spmm.plan_create(64, K, *arrays, tiles=32)
    assert plan.describe()["tile_rows"] == 32
    assert right(torch_gpu, plan, K, *arrays)


@pytest.mark.parametrize("K", [20000, 65536, 70000])
def test_columns_outside_are_found(torch_gpu, K):  # noqa: F811
    row_ptr, col_idx, vals = matrix(SMALLEST + 5, K, 1)
    for at in (0, SMALLEST // 2, SMALLEST + 4):
        for outside in (-1, K, K + 65536, -65536, 2 ** 31 - 1):
            bad = col_idx.copy()
            bad[at] = outside
            with pytest.raises(spmm.SpmmError) as err:
                spmm.plan_create(64, K, row_ptr, bad, vals, tiles=32)
            assert err.value.status == spmm.SPMM_ERR_INVALID_CSR
    plan = spmm.plan_create(64, K, row_ptr, col_idx, vals, tiles=32)   # the memory was given back
    assert right(torch_gpu, plan, K, row_ptr, col_idx, vals)


def test_creations_at_the_same_time(torch_gpu):  # noqa: F811
    """One of them has the memory, the others upload as small matrices do."""
    cases = [(K, matrix(600000 + i, K, i)) for i, K in enumerate((20000, 65536, 70000, 30000))]
    plans = [None] * len(cases)

    def create(i):
        for _ in range(5):
            plans[i] = spmm.plan_create(64, cases[i][0], *cases[i][1], tiles=32)

    threads = [threading.Thread(target=create, args=(i,)) for i in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for plan, (K, arrays) in zip(plans, cases):
        assert right(torch_gpu, plan, K, *arrays)


def mapped():
    """Bytes of this process's mappings of the device's memory: pinned memory and what the device has allocated."""
    total = 0
    with open("/proc/self/maps") as f:
        for line in f:
            if "/dev/dri/" in line:
                first, last = line.split()[0].split("-")
                total += int(last, 16) - int(first, 16)
    return total


def test_the_pinned_memory_is_given_back(torch_gpu):  # noqa: F811
    """With the last plan on tiles, also right after it was made, and after a creation that failed; 6 MiB of it while there is one."""
    K = 20000
    row_ptr, col_idx, vals = matrix(SMALLEST + 5, K, 1)
    outside = col_idx.copy()
    outside[9] = K
    small = spmm.plan_create(64, K, *matrix(4096, K, 2), tiles=32)   # what the library and the runtime set up once
    del small
    gc.collect()
    torch_gpu.cuda.synchronize()
    before = mapped()
    with pytest.raises(spmm.SpmmError):
        spmm.plan_create(64, K, row_ptr, outside, vals, tiles=32)
    assert mapped() == before
    for _ in range(2):
        first = spmm.plan_create(64, K, row_ptr, col_idx, vals, tiles=32)
        second = spmm.plan_create(64, K, row_ptr, col_idx, vals, tiles=32)
        with_two = mapped()
        del first
        with_one = mapped()
        del second
        assert mapped() == before
        assert with_one - before >= 6 << 20 and with_two > with_one
