"""The native tensor-level entry behind Plan.execute (GPU machine only)."""
import sys
import threading
import time

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


def test_other_threads_run_during_a_call(torch_gpu):  # noqa: F811
    """With the interpreter's own switching out of the way, another thread comes to run only where a call
    lets go of the interpreter."""
    torch = torch_gpu
    plan = one_column_plan(256)
    B = torch.ones((1, 32), device="cuda")
    C = plan.execute(B)
    ready, stop, turns = threading.Event(), threading.Event(), [0]

    def other():
        ready.set()
        while not stop.is_set():
            turns[0] += 1
            time.sleep(0)   # hand the interpreter back

    interval = sys.getswitchinterval()
    thread = threading.Thread(target=other)
    thread.start()
    ready.wait()
    sys.setswitchinterval(1000.0)
    try:
        time.sleep(0.05)   # the other thread's wait is one of the new interval from here on
        ran = 0
        for _ in range(2000):
            before = turns[0]
            plan.execute(B, C)
            ran += turns[0] != before
    finally:
        sys.setswitchinterval(interval)
        stop.set()
        thread.join()
        torch.cuda.synchronize()
    print("the other thread ran during %d of 2000 calls" % ran)
    assert ran > 0
