"""The structures of the boundary grow at their end: callers with fewer fields than the library, or with more."""
import ctypes

import numpy as np
import pytest

import paper_2506_15174_amd as spmm
from paper_2506_15174_amd.binding import Options, PlanInfo

GUARD = 0x5A5A5A5A


@pytest.fixture
def lib():
    lib = ctypes.CDLL(spmm.load()._name)   # a handle of its own: no argument types set by the binding
    return lib


def create(lib, words, size=None, function="spmm_plan_create_sized"):
    """A 3 x 4 matrix with the options given as 32-bit words; (status, handle)."""
    row_ptr, col_idx = np.array([0, 2, 2, 3], np.int32), np.array([0, 3, 1], np.int32)
    vals, opts, handle = np.ones(3, np.float32), np.array(words, np.uint32), ctypes.c_void_p(1)
    args = [ctypes.byref(handle), ctypes.c_int64(3), ctypes.c_int64(4)] + \
        [ctypes.c_void_p(x.ctypes.data) for x in (row_ptr, col_idx, vals, opts)]
    if size is not None:
        args.append(ctypes.c_size_t(size))
    return getattr(lib, function)(*args), handle


def words_of(**fields):
    return np.frombuffer(bytes(Options(**fields)), np.uint32).copy()


def test_programs_compiled_before_the_last_fields(lib):
    """The functions without a size end where their last callers' structures ended."""
    opts = words_of(host_only=1, tiles=99)   # 99 stands for what lies behind the caller's structure
    assert Options.tiles.offset == 4 * (len(opts) - 1)
    st, plan = create(lib, opts, function="spmm_plan_create_ex")
    assert st == spmm.SPMM_OK
    out = np.full(ctypes.sizeof(PlanInfo) // 4, GUARD, np.uint32)
    assert lib.spmm_plan_describe(plan, ctypes.c_void_p(out.ctypes.data)) == spmm.SPMM_OK
    end = PlanInfo.tile_rows.offset // 4
    assert (out[end:] == GUARD).all() and list(out[:6:2]) == [3, 4, 3] and out[end - 2] == 4
    lib.spmm_plan_destroy(plan)


@pytest.mark.parametrize("fields", [0, 3, 13, 14, 20])
def test_fewer_options_than_the_library_and_more(lib, fields):
    opts = np.concatenate([words_of(host_only=1, ufi=4, tiles=99), np.zeros(8, np.uint32)])
    st, plan = create(lib, opts, 4 * fields)
    if fields > 13:
        assert st == spmm.SPMM_ERR_INVALID_ARG and plan.value is None   # the 99 counts
        opts[13] = 0
        st, plan = create(lib, opts, 4 * fields)
    if fields == 0:   # nothing of it is read: no host_only, which needs a device
        assert st in (spmm.SPMM_OK, spmm.SPMM_ERR_HIP)
    else:
        assert st == spmm.SPMM_OK
        out = np.full(50, GUARD, np.uint32)
        assert lib.spmm_plan_describe_sized(plan, ctypes.c_void_p(out.ctypes.data), ctypes.c_size_t(4 * 40)) == spmm.SPMM_OK
        known = ctypes.sizeof(PlanInfo) // 4
        assert known < 40 and (out[known:40] == 0).all() and (out[40:] == GUARD).all()
        assert out[6] == (4 if fields > 3 else out[6])
        few = np.full(50, GUARD, np.uint32)
        assert lib.spmm_plan_describe_sized(plan, ctypes.c_void_p(few.ctypes.data), ctypes.c_size_t(24)) == spmm.SPMM_OK
        assert (few[:6] == out[:6]).all() and (few[6:] == GUARD).all()
    lib.spmm_plan_destroy(plan)


def test_an_option_the_library_does_not_know_is_refused(lib):
    opts = np.concatenate([words_of(host_only=1), np.zeros(2, np.uint32)])
    opts[15] = 1
    st, plan = create(lib, opts, 64)
    assert st == spmm.SPMM_ERR_UNSUPPORTED and plan.value is None
    st, plan = create(lib, opts, 60)
    assert st == spmm.SPMM_OK
    lib.spmm_plan_destroy(plan)
