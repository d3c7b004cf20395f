"""The native tensor-level entry behind Plan.execute (GPU machine only)."""
import numpy as np
import pytest

import paper_2506_15174_amd as spmm

from test_gpu_parity import torch_gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def one_column_plan(M):
    """A of M x 1, all ones: C repeats the row of B."""
    return spmm.plan_create(M, 1, np.arange(M + 1), np.zeros(M), np.ones(M))


def test_no_memory_for_the_output_is_torchs_own_error(torch_gpu):  # noqa: F811
    """An output of 1 TiB: the allocator's error type, which callers catch to try a smaller batch."""
    torch = torch_gpu
    plan = one_column_plan(1 << 20)
    B = torch.ones((1, 1 << 18), device="cuda")
    with pytest.raises(torch.cuda.OutOfMemoryError):
        plan.execute(B)
    assert torch.equal(plan.execute(B[:, :4].contiguous()), torch.ones((1 << 20, 4), device="cuda"))
