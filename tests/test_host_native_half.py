"""The device calls without the native half of the binding, or with one that was built for another torch: ctypes makes them."""
import shutil
import warnings

import pytest
import torch

import paper_2505_10183_amd as kt
from paper_2505_10183_amd import binding


@pytest.fixture
def unloaded(monkeypatch):
    """The binding as it is before its first device call."""
    kt.binding.lib()
    for name, value in (("_native_of", {}), ("_calls", None), ("_marshal", None)):
        monkeypatch.setattr(binding, name, value, raising=False)
    return monkeypatch


def refused(plan, tensors):
    """A call that the library refuses (bucket 5 of 1): it got there."""
    with pytest.raises(kt.KtError, match="bucket 5 outside") as e:
        plan.kt_bucket_pack(5, tensors, [torch.zeros(64)], 0)
    assert e.type is kt.KtError


def calls(expect_warning):
    plan = kt.Plan([5, 7], "f32", 0, 16)
    t = [torch.zeros(5), torch.zeros(7)]
    for form in (t, [x.data_ptr() for x in t], plan.marshal(t)):
        with warnings.catch_warnings(record=True) as got:
            warnings.simplefilter("always")
            refused(plan, form)
        assert [w.category for w in got] == ([RuntimeWarning] if expect_warning else [])
        expect_warning = False          # once in a process
    return plan


def test_the_native_half_is_used_where_it_was_built_for_this_torch(unloaded):
    assert calls(False)._calls is not None


def test_without_it(unloaded, tmp_path):
    unloaded.setattr(binding, "MARSHAL_PATH", str(tmp_path / "_kt_marshal.so"))
    assert calls(True)._calls is None


@pytest.mark.parametrize("version", ["2.9.0", torch.__version__ + "1", torch.__version__[:-1], ""])
def test_built_for_another_torch(unloaded, tmp_path, version):
    path = str(tmp_path / "_kt_marshal.so")
    shutil.copy(binding.MARSHAL_PATH, path)
    unloaded.setattr(binding, "MARSHAL_PATH", path)
    unloaded.setattr(torch, "__version__", version)
    assert calls(True)._calls is None
