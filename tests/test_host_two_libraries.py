"""Two copies of libkt.so loaded in one process (as bench.py --ab has them): a plan's calls stay with the library that made it."""
import shutil

import pytest
import torch

import paper_2505_10183_amd as kt
from paper_2505_10183_amd import binding


@pytest.fixture
def second(tmp_path):
    """The library that the binding holds, and a copy of it loaded beside it."""
    first, path = binding.lib(), binding.LIB_PATH
    copy = str(tmp_path / "libkt_copy.so")
    shutil.copy(path, copy)
    binding._lib, binding.LIB_PATH = None, copy
    try:
        other = binding.lib()
    finally:
        binding._lib, binding.LIB_PATH = first, path
    assert other._handle != first._handle
    yield first, other
    binding._lib = first


FORMS = {"lists": lambda plan, l: l, "marshalled": lambda plan, l: plan.marshal(l), "addresses": lambda plan, l: [t.data_ptr() for t in l]}


def plan_of(library):
    binding._lib = library
    return kt.Plan([5, 7, 3], "f32", 0, 16)


def refused_calls(plan, form):
    """Every device call of the binding with a bucket that the plan does not have: no GPU is touched."""
    made = lambda n: FORMS[form](plan, [torch.zeros(8) for _ in range(n)])
    T, b, s = made(3), made(1), 0
    yield lambda: plan.kt_bucket_pack(5, T, b, s)
    yield lambda: plan.kt_weighted_reduce(5, made(2), 2, [0.5, 0.5], b, s)
    yield lambda: plan.kt_bucket_unpack_scale(5, b, 1.0, T, s)
    yield lambda: plan.kt_fused_step(5, T, b, 2, [0.5, 0.5], 1.0, T, s)
    yield lambda: plan.kt_bucket_unpack_sgd(5, b, 1.0, T, T, 0.1, 0.9, 0.0, False, s)
    yield lambda: plan.kt_bucket_unpack_sgd_master(5, b, 1.0, T, T, T, 0.1, 0.9, 0.0, False, s)
    yield lambda: plan.kt_fused_step_sgd(5, T, b, 2, [0.5, 0.5], 1.0, T, T, None, 0.1, 0.9, 0.0, False, s)
    yield lambda: plan.kt_fused_step_noalloc(5, T, b, 2, [0.5, 0.5], 1.0, T, s)
    yield lambda: plan.kt_weighted_reduce(5, made(65), 65, [0.5] * 65, b, s)       # K that no library takes


@pytest.mark.parametrize("form", ["lists", "marshalled", "addresses"])
@pytest.mark.parametrize("current", [0, 1])
def test_a_plan_calls_the_library_that_made_it(second, current, form):
    plans = [plan_of(L) for L in second]
    binding._lib = second[current]
    for which in (0, 1, 0):
        plan, own, other = plans[which], second[which], second[1 - which]
        for call in refused_calls(plan, form):
            # the message of the last call is the library's: a call that goes astray leaves the other one's changed
            assert other.kt_plan_shares(None, 0, 1, None, None) != 0
            before = other.kt_last_error()
            with pytest.raises(kt.KtError) as e:
                call()
            assert e.value.args and own.kt_last_error() and own.kt_last_error().decode() in str(e.value)
            assert own.kt_last_error() != before and other.kt_last_error() == before
    for p in plans:
        assert p.num_tensors == 3 and p.num_tiles == 1 and p.bucket_info(0)[2] == 3 and p.tensor_info(2)[0] == 0
        p.close()
