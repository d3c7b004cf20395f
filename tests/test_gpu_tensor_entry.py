"""The native tensor-level entry behind Plan.execute (needs the GPU)."""
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


def test_what_the_entry_refuses(torch_gpu):  # noqa: F811
    """The errors that the entry has raised since it was written in Python, by type."""
    torch = torch_gpu
    plan = spmm.plan_create(3, 2, [0, 1, 1, 2], [0, 1], [1.0, 2.0])
    B, C = torch.ones((2, 5), device="cuda"), torch.empty((3, 5), device="cuda")
    want = torch.tensor([[1.0], [0.0], [2.0]], device="cuda").expand(3, 5)
    assert torch.equal(plan.execute(B), want) and plan.execute(B, C) is C and torch.equal(C, want)
    wrong_B = [torch.ones((2, 5)), B.double(), B.half(), torch.ones((5, 2), device="cuda").t(), torch.ones((2, 10), device="cuda")[:, ::2],
               torch.ones(10, device="cuda"), torch.ones((1, 2, 5), device="cuda"), torch.ones((3, 5), device="cuda")]
    for bad in wrong_B:
        with pytest.raises(ValueError, match="B "):
            plan.execute(bad)
    wrong_C = [torch.empty((3, 5)), C.double(), torch.empty((5, 3), device="cuda").t(), torch.empty((3, 4), device="cuda"),
               torch.empty((4, 5), device="cuda"), torch.empty(15, device="cuda")]
    for bad in wrong_C:
        with pytest.raises(ValueError, match="C must"):
            plan.execute(B, bad)
    for bad in (np.ones((2, 5), np.float32), [[1.0]], 3):
        with pytest.raises(TypeError):
            plan.execute(bad)
        with pytest.raises(TypeError):
            plan.execute(B, bad)
    with pytest.raises(AttributeError):
        plan.execute(B, stream=7)
    with pytest.raises(spmm.SpmmError) as err:   # N = 0
        plan.execute(torch.ones((2, 0), device="cuda"))
    assert err.value.status == spmm.SPMM_ERR_INVALID_ARG
    grad = B.clone().requires_grad_()
    assert not plan.execute(grad).requires_grad
    plan.destroy()
    plan.destroy()
    with pytest.raises(spmm.SpmmError) as err:
        plan.execute(B, C)
    assert err.value.status == spmm.SPMM_ERR_INVALID_ARG
    host = spmm.plan_create(3, 2, [0, 1, 1, 2], [0, 1], [1.0, 2.0], host_only=True)
    with pytest.raises(spmm.SpmmError) as err:
        host.execute(B, C)
    assert err.value.status == spmm.SPMM_ERR_INVALID_ARG


def test_the_output_on_a_side_stream(torch_gpu):  # noqa: F811
    torch = torch_gpu
    plan = one_column_plan(1000)
    B = torch.arange(32.0, device="cuda").reshape(1, 32)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    given = plan.execute(B, torch.empty((1000, 32), device="cuda"), stream=side)
    with torch.cuda.stream(side):
        made = plan.execute(B)
    side.synchronize()
    assert torch.equal(given, B.expand(1000, 32)) and torch.equal(made, B.expand(1000, 32))
