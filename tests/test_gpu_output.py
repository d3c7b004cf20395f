"""The output that Plan.execute allocates: like torch.empty's in every setting that torch.empty knows of.  Needs the GPU."""
import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from workloads import generators as gen
from test_gpu_parity import torch_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [0, 1, 65])
def test_the_output_is_what_torch_empty_would_make(torch_gpu, M):  # noqa: F811
    torch = torch_gpu
    from torch.utils._python_dispatch import TorchDispatchMode
    csr = gen.uniform_positions(M, 40, 0.5, 1) if M else gen.Csr(0, 40, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))
    plan = spmm.plan_create(M, 40, csr.row_ptr, csr.col_idx, csr.vals)
    B = torch.randn(40, 9, device="cuda", requires_grad=True)
    A = torch.zeros(M, 40, dtype=torch.float64)
    for i in range(M):
        A[i, torch.from_numpy(csr.col_idx[csr.row_ptr[i]:csr.row_ptr[i + 1]]).long()] = torch.from_numpy(csr.vals[csr.row_ptr[i]:csr.row_ptr[i + 1]]).double()
    ref = (A @ B.detach().cpu().double()).numpy()

    def check(C):
        like = torch.empty((M, 9), device=B.device)
        assert (C.shape, C.stride(), C.dtype, C.device, C.requires_grad, C.is_inference(), C.layout) == \
               (like.shape, like.stride(), like.dtype, like.device, like.requires_grad, like.is_inference(), like.layout)
        assert C.grad_fn is None and C.storage_offset() == 0 and C.untyped_storage().nbytes() == like.untyped_storage().nbytes()
        torch.cuda.synchronize()
        assert np.allclose(C.detach().cpu().numpy(), ref, atol=1e-5)
        return C

    C = check(plan.execute(B))
    C.add_(1.0)                                  # an ordinary tensor: changed in place, differentiated through
    (C.requires_grad_().sum() * 2).backward()
    assert bool((C.grad == 2).all())
    with torch.no_grad():
        check(plan.execute(B))
    with torch.inference_mode():
        check(plan.execute(B))
    seen = []

    class Watch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(str(func))
            return func(*args, **(kwargs or {}))

    with Watch():
        C = plan.execute(B)
    check(C)
    assert any("empty" in name for name in seen)
    before = torch.are_deterministic_algorithms_enabled()
    torch.use_deterministic_algorithms(True)
    try:
        check(plan.execute(B))
    finally:
        torch.use_deterministic_algorithms(before)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]) as prof:
        C = plan.execute(B)
    check(C)
    assert any("empty" in e.key for e in prof.key_averages())
